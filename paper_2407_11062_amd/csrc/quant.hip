// HBM-bound passes: min/max initialisation, the quantize pass (Eq.(1) -> packed N-bit codes),
// zero-point packing / unpacking, code unpacking, and the small reductions the GEMM epilogues need.
#include "common.h"
#include "kernels.h"

namespace eqat {

// ---------------------------------------------------------------------------------------------
// Eq.(1) for one weight.  The code must equal clamp(round_half_even(fl32(w/s)) + zbar, 0, Qmax) exactly.  The exact
// quotient costs a dozen instructions, so k_quantize first rounds w * r for an r just below and one just above 1/s (2^-21
// relative, where the reciprocal is within 2^-23 and the quotient's own rounding 2^-24): rounding is monotonic, so where both
// give the same integer, fl32(w/s) gives it too.  A chunk in which some weight's differ is redone with this exact division.
__device__ __forceinline__ float quant_exact(float w, float s) { return __builtin_rintf(w / s); }

template <typename WT> struct Chunk8;   // 8 consecutive weights of one lane
template <> struct Chunk8<bf16_t> {
    static constexpr int kBytes = 16;
    uintx4 v;
    template <bool ONCE = false> __device__ __forceinline__ void load(const bf16_t *p)          // ONCE: past the caches
    {
        const uintx4 *const q = reinterpret_cast<const uintx4 *>(p);
        v = ONCE ? __builtin_nontemporal_load(q) : *q;
    }
    __device__ __forceinline__ float get(int k) const
    {
        const uint32_t u = v[k >> 1];
        return __uint_as_float((k & 1) ? (u & 0xFFFF0000u) : (u << 16));
    }
};
template <> struct Chunk8<float> {
    static constexpr int kBytes = 32;
    floatx4 a, b;
    template <bool ONCE = false> __device__ __forceinline__ void load(const float *p)            // (32 bytes a lane: never past the caches)
    {
        a = *reinterpret_cast<const floatx4 *>(p);
        b = *reinterpret_cast<const floatx4 *>(p + 4);
    }
    // Past the caches, neighbouring lanes neighbouring 16 bytes, twice: lanes 2 i and 2 i + 1 the halves of chunk i and those of chunk 32 + i of the wave, of which
    // the even lane then keeps the first and the odd one the second.
    __device__ __forceinline__ void load_halves(const float *p, const float *q)
    {
        a = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(p));
        b = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(q));
    }
    __device__ __forceinline__ void exchange(bool odd)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int mine = __float_as_int(odd ? a[k] : b[k]);
            const float theirs = __int_as_float(__builtin_amdgcn_update_dpp(0, mine, 0xB1, 0xF, 0xF, false));      // quad_perm [1,0,3,2]
            a[k] = odd ? theirs : a[k];
            b[k] = odd ? b[k] : theirs;
        }
    }
    __device__ __forceinline__ float get(int k) const { return k < 4 ? a[k] : b[k - 4]; }
};

__device__ __forceinline__ uint32_t quad_bcast(uint32_t v, int k)
{
    // value of lane (lane & ~3) + k, through a DPP quad permute
    switch (k) {
    case 0: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x00, 0xF, 0xF, false);
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x55, 0xF, 0xF, false);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xAA, 0xF, 0xF, false);
    default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xFF, 0xF, 0xF, false);
    }
}

// Place of the code k of a lane's eight: bit 3 k of the dense stream (2, 4 k); in the working layout byte k % 4, field k / 4.
template <bool WORK, int BITS> __host__ __device__ constexpr int code_place(int k) { return WORK ? 8 * (k % 4) + WorkCodes<BITS>::kField * (k / 4) : k * BITS; }
// the same word at all eight places, added up
template <bool WORK, int BITS> __host__ __device__ constexpr uint32_t packed_sum(uint32_t v)
{
    uint32_t p = 0;
    for (int k = 0; k < 8; ++k) p += v << code_place<WORK, BITS>(k);
    return p;
}
// From here on floats are integers, and what is added to it is rounded to one, ties to even: the low bits of kIntegers + n are n.
constexpr float kIntegers = 0x1.8p23f;

// Bit k: a[k] is not b[k], as words.  A compare and an add with carry (bits = 2 bits + carry) each; two wait states lie between a vector instruction that writes
// a scalar register and one that reads it, which the compiler does not put into assembly: three carries take turns, so that other compares and sums lie there.
__device__ __forceinline__ uint32_t differ_bits(const float (&a)[8], const float (&b)[8])
{
    uint32_t bits = 0;
    uint64_t c0, c1, c2;
    asm("v_cmp_ne_u32_e64 %1, %11, %19\n\t"
        "v_cmp_ne_u32_e64 %2, %10, %18\n\t"
        "v_cmp_ne_u32_e64 %3, %9, %17\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\t"
        "v_cmp_ne_u32_e64 %1, %8, %16\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
        "v_cmp_ne_u32_e64 %2, %7, %15\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\t"
        "v_cmp_ne_u32_e64 %3, %6, %14\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\t"
        "v_cmp_ne_u32_e64 %1, %5, %13\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
        "v_cmp_ne_u32_e64 %2, %4, %12\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2"
        : "+&v"(bits), "=&s"(c0), "=&s"(c1), "=&s"(c2)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]),
          "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(b[6]), "v"(b[7]) : "vcc");
    return bits;
}

// The quantize pass.  One lane owns 8 consecutive weights (a 16- or 32-byte load); the four lanes of a
// quad own one 32-code segment, i.e. BITS output words, assembled with quad permutes.
//   codes     [O, I*BITS/32] words      packed stream (same layout as eqat_pack's Wpacked)
//   clampbits [O, I/8] bytes (CLAMPBITS) bit k of byte e/8: weight e was clamped by Eq.(1)
//   sz        [O, G] float2 or NULL     (s, zbar) per group, zbar = clamp(round(z), 0, Qmax)
// Rows are contiguous and g divides I, so weight e belongs to group e / g of the flattened [O*G] arrays.
// Per weight the common path costs six instructions: widen, two fused multiply-adds that round to an integer (kIntegers + zbar is
// added; a tie, which an odd zbar would turn the other way, is a chunk for the exact path), their comparison, the clamp, a shift-add of the
// float as it is (the exponents of all eight add up to a constant).  With the clamp plane two more.  With the ten there were before (multiply,
// round, difference, maximum, clamp, conversion, shift-add, and three for the clamp plane) the pass was bound by its arithmetic: seven matrices of a
// 4096 / 11008 block, bf16, quantize 99 -> 94 us, and 84 with W loaded past the caches (see kQuantizeOnceBytes); pack 94 -> 86, where the end of W
// comes from the memory-side cache and such loads lose 1-3 %.  fp32 weights gain by them only where neighbouring lanes read neighbouring 16 bytes
// (load_halves; 810 MB, 4 bit: 187 -> 158 us, without that 192); through the caches the exchange behind that costs 0.2 to 0.7 us of a launch (quantize and forward, 238 tokens, 352 -> 7000
// 14.1 / 14.6, 136 tokens, 4608 -> 1936 30.8 / 31.5; level from 100 MB on).
// WORK = false: the dense stream of the C ABI (eqat_pack).  WORK = true: the library's working layout (WorkCodes).
// Zero points at N bits: one thread per output word (tail bits of a row are zero).
template <int BITS>
__device__ __forceinline__ void pack_z_word(const float *__restrict__ z, uint32_t *__restrict__ zpacked, uint32_t t,
                                            uint32_t G, uint32_t row_words)
{
    const uint32_t row = t / row_words, w = t - row * row_words;
    constexpr float qmax = (float)((1 << BITS) - 1);
    const uint32_t bit0 = w * 32u;
    uint32_t j = bit0 / BITS;                   // first code with bits in this word
    uint64_t acc = 0;
    for (; j < G && j * BITS < bit0 + 32u; ++j) {
        const uint32_t code = (uint32_t)zbar_of(z[row * G + j], qmax);
        const int sh = (int)(j * BITS) - (int)bit0;         // may be negative for a code straddling in from the left
        acc |= sh >= 0 ? ((uint64_t)code << sh) : ((uint64_t)code >> (-sh));
    }
    zpacked[t] = (uint32_t)acc;
}

struct QuantizeArgs {
    const void *W; const float *s, *z;
    uint32_t *codes; uint8_t *clampbits; floatx2 *sz;
    uint32_t n_chunks, g; int g_shift;
    // eqat_pack only: the blocks past n_quant_blocks pack the zero points (one thread per word)
    uint32_t *zpacked; uint32_t n_quant_blocks, n_zwords, G, row_words;
    // words the launch clears on the side (arrival counters of the GEMM launches that follow); NULL: none
    uint32_t *zero_words; uint32_t n_zero;
};

// block / nblocks: this workgroup's number among those that share the job
__device__ __forceinline__ void clear_words(uint32_t *__restrict__ w, uint32_t n, uint32_t block, uint32_t nblocks)
{
    for (uint32_t i = block * blockDim.x + threadIdx.x; i < n; i += nblocks * blockDim.x) w[i] = 0u;
}

// Up to kMaxBatch matrices in one launch (the linears of a decoder block are 34-90 MB each at 7B size: alone, each would
// be a 10-25 us launch that spends a good part of its time filling and draining the chip).  Workgroups
// [first[i], first[i + 1]) work on matrix i.
struct QuantizeBatch { QuantizeArgs a[kMaxBatch]; uint32_t first[kMaxBatch + 1]; };
__device__ __forceinline__ int batch_slot(const uint32_t (&first)[kMaxBatch + 1], uint32_t block)
{
    int i = 0;
#pragma unroll
    for (int k = 1; k < kMaxBatch; ++k) i += block >= first[k] ? 1 : 0;      // first[k] of unused slots: the grid size
    return i;
}

constexpr int kQuantUnroll = 4;     // chunks per thread: 64 B (bf16) / 128 B (fp32) of W in flight per lane
// eqat_pack of one large bf16 matrix (the 70B-sized ones, 235 M weights): twice the loads in flight measured +5 %; on
// smaller matrices, with several matrices per launch and in the working-layout instantiations it measured 2-10 % slower.
constexpr int kPackUnrollLarge = 8;
constexpr size_t kPackLargeChunks = (size_t)1 << 24;     // 8-weight chunks: 134 M weights

// ONCE: W is loaded past the caches
template <typename WT, int BITS, bool CLAMPBITS, bool WORK, bool ONCE = false, int U = kQuantUnroll>
__global__ __launch_bounds__(256) void k_quantize(const QuantizeBatch batch)
{
    // Packing walks its matrices from the last weight to the first: the pass that comes before it (min/max, an optimizer
    // step) leaves the end of W in the 256 MB memory-side cache, not the beginning.  Eight blocks at a time, so that every
    // weight stays with the XCD, and the L2, that it was on (min/max + pack of 4096 x 1024 in fp32: 13.2 -> 12.0 us; front to back 12.0).
    const uint32_t whole = gridDim.x & ~7u;
    const uint32_t bid = WORK || blockIdx.x >= whole ? blockIdx.x : whole - 8u - (blockIdx.x & ~7u) + (blockIdx.x & 7u);
    const int slot = batch_slot(batch.first, bid);
    const QuantizeArgs &a = batch.a[slot];
    const uint32_t block = bid - batch.first[slot];
    if (a.zero_words != nullptr) clear_words(a.zero_words, a.n_zero, block, batch.first[slot + 1] - batch.first[slot]);
    if (block >= a.n_quant_blocks) {
        const uint32_t t = (block - a.n_quant_blocks) * 256u + threadIdx.x;
        if (t < a.n_zwords) pack_z_word<BITS>(a.z, a.zpacked, t, a.G, a.row_words);
        return;
    }
    const WT *__restrict__ W = reinterpret_cast<const WT *>(a.W);
    constexpr float qmax = (float)((1 << BITS) - 1);
    constexpr bool SPREAD = ONCE && sizeof(WT) == 4;
    const uint32_t first = block * (256u * U) + (threadIdx.x & ~63u), lane = threadIdx.x & 63u;
    // chunk index; n_chunks % 4 == 0 so quads stay whole
    const uint32_t c0 = first + (SPREAD ? (lane >> 1) + 32u * (lane & 1u) : lane);
    // all loads of the thread's U chunks first: the pass lives on bytes in flight
    Chunk8<WT> ch[U];
    uint32_t gi[U];
    float sv[U], zb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t c = c0 + u * 256u;
        const uint32_t cc = c < a.n_chunks ? c : 0u;             // past the end: recompute chunk 0, store nothing
        const uint32_t e = cc * 8u;
        gi[u] = a.g_shift >= 0 ? (e >> a.g_shift) : (e / a.g);
        if constexpr (SPREAD) {
            const uint32_t p0 = (first + u * 256u) * 2u + lane, p1 = p0 + 64u, n = a.n_chunks * 2u;     // pieces of four weights
            ch[u].load_halves(W + (size_t)(p0 < n ? p0 : 0u) * 4, W + (size_t)(p1 < n ? p1 : 0u) * 4);
        } else ch[u].template load<ONCE>(W + e);
        sv[u] = a.s[gi[u]];
        zb[u] = a.z[gi[u]];
    }
    if constexpr (SPREAD) {
#pragma unroll
        for (int u = 0; u < U; ++u) ch[u].exchange((lane & 1u) != 0);
    }
    const uint32_t q4 = c0 & 3u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t c = c0 + u * 256u;
        if (c >= a.n_chunks) break;
        const uint32_t e = c * 8u;
        const float zbar = zbar_of(zb[u], qmax);
        if (a.sz != nullptr && e == gi[u] * a.g) { floatx2 o; o[0] = sv[u]; o[1] = zbar; a.sz[gi[u]] = o; }
        const float rinv = __builtin_amdgcn_rcpf(sv[u]);          // 1 ulp; s is a normal number
        const float below = rinv * (1.0f - 0x1p-21f), above = rinv * (1.0f + 0x1p-21f), base = kIntegers + zbar;
        float f[8];
        uint32_t differ = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float w = ch[u].get(k), other = __builtin_fmaf(w, above, base);
            f[k] = __builtin_fmaf(w, below, base);
            differ |= __float_as_uint(f[k]) ^ __float_as_uint(other);
            asm("" : "+v"(differ));                                // one v_bitop3 a weight, not a comparison and two selects
        }
        if (differ != 0) {
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = quant_exact(ch[u].get(k), sv[u]) + base;
        }
        float fc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) fc[k] = __builtin_amdgcn_fmed3f(f[k], kIntegers, kIntegers + qmax);
        if constexpr (CLAMPBITS) {
            a.clampbits[c] = (uint8_t)differ_bits(f, fc);
        }
        // the codes at their places in a word
        uint32_t p = 0u - packed_sum<WORK, BITS>(__builtin_bit_cast(uint32_t, kIntegers));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            p += __float_as_uint(fc[k]) << code_place<WORK, BITS>(k);
            asm("" : "+v"(p));                                     // one v_lshl_add a weight
        }
        if constexpr (!WORK) {
            const uint32_t p0 = quad_bcast(p, 0), p1 = quad_bcast(p, 1), p2 = quad_bcast(p, 2), p3 = quad_bcast(p, 3);
            uint32_t word;
            if constexpr (BITS == 2) {
                word = (q4 == 0) ? (p0 | (p1 << 16)) : (p2 | (p3 << 16));
            } else if constexpr (BITS == 3) {
                word = (q4 == 0) ? (p0 | (p1 << 24)) : (q4 == 1) ? ((p1 >> 8) | (p2 << 16)) : ((p2 >> 16) | (p3 << 8));
            } else {
                word = (q4 == 0) ? p0 : (q4 == 1) ? p1 : (q4 == 2) ? p2 : p3;
            }
            if (q4 < (uint32_t)BITS) a.codes[(c >> 2) * BITS + q4] = word;
        } else {
            if constexpr (BITS == 2) {
                const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)p, SPREAD ? 0x4E : 0xB1, 0xF, 0xF, false);   // the chunk beside this one: quad_perm [2,3,0,1] or [1,0,3,2]
                if ((q4 & 1u) == 0) a.codes[(c >> 2) * 2 + (q4 >> 1)] = p | (other << 4);
            } else {
                a.codes[c] = p;
            }
        }
    }
}

// The dense stream of the C ABI -> the working layout (one thread per 32-code segment).
template <int BITS>
__device__ __forceinline__ void repack_segment(const uint32_t *__restrict__ packed, uint32_t *__restrict__ work, uint32_t t)
{
    uint32_t in[BITS];
#pragma unroll
    for (int k = 0; k < BITS; ++k) in[k] = packed[(size_t)t * BITS + k];
    uint32_t out[WorkCodes<BITS>::kWords] = {};
#pragma unroll
    for (int e = 0; e < 32; ++e)
        out[WorkCodes<BITS>::word_of(e)] |= code_at_rt<BITS>(in, e) << WorkCodes<BITS>::bit_of(e);
#pragma unroll
    for (int k = 0; k < WorkCodes<BITS>::kWords; ++k) work[(size_t)t * WorkCodes<BITS>::kWords + k] = out[k];
}

// (s, z) pair of group t for the E2E-QP kernels: z from the packed N-bit zero points, or from a float array.
// zb_out (may be NULL) also receives the zero point alone; sz may be NULL when only that is wanted.
template <int BITS>
__device__ __forceinline__ void pair_sz(const float *__restrict__ s, const uint32_t *__restrict__ zpacked,
                                        const float *__restrict__ zfloat, floatx2 *__restrict__ sz, float *__restrict__ zb_out,
                                        uint32_t t, uint32_t G, uint32_t row_words)
{
    float zv;
    if (zfloat != nullptr) {
        zv = zfloat[t];
    } else {
        const uint32_t row = t / G, j = t - row * G;
        const uint32_t bit = j * BITS, wi = bit >> 5, sh = bit & 31u;
        uint64_t two = zpacked[row * row_words + wi];
        if (sh + BITS > 32u) two |= (uint64_t)zpacked[row * row_words + wi + 1] << 32;
        zv = (float)((uint32_t)(two >> sh) & ((1u << BITS) - 1u));
    }
    if (zb_out != nullptr) zb_out[t] = zv;
    if (sz != nullptr) { floatx2 o; o[0] = s[t]; o[1] = zv; sz[t] = o; }
}

// What an E2E-QP call needs before its GEMMs, in one launch: the first n_repack_blocks workgroups re-lay the codes from
// the dense stream into the working layout (packed == NULL: none; a prepared layer has them already), the rest write the
// (s, z) pairs (and / or the zero points alone: what eqat_qlinear_prepare keeps).
template <int BITS>
__global__ __launch_bounds__(256) void k_e2e_prepare(const uint32_t *__restrict__ packed, uint32_t *__restrict__ work,
                                                     uint32_t n_segs, uint32_t n_repack_blocks,
                                                     const float *__restrict__ s, const uint32_t *__restrict__ zpacked,
                                                     const float *__restrict__ zfloat, floatx2 *__restrict__ sz,
                                                     float *__restrict__ zb_out, uint32_t n_groups, uint32_t G,
                                                     uint32_t row_words, uint32_t *__restrict__ zero_words, uint32_t n_zero)
{
    if (zero_words != nullptr) clear_words(zero_words, n_zero, blockIdx.x, gridDim.x);
    if (blockIdx.x < n_repack_blocks) {
        const uint32_t t = blockIdx.x * 256u + threadIdx.x;
        if (t < n_segs) repack_segment<BITS>(packed, work, t);
    } else {
        const uint32_t t = (blockIdx.x - n_repack_blocks) * 256u + threadIdx.x;
        if (t < n_groups) pair_sz<BITS>(s, zpacked, zfloat, sz, zb_out, t, G, row_words);
    }
}

template <int BITS>
__global__ __launch_bounds__(256) void k_unpack_codes(const uint32_t *__restrict__ packed, int32_t *__restrict__ out,
                                                      uint32_t n_segs)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= n_segs) return;
    uint32_t w[BITS];
#pragma unroll
    for (int k = 0; k < BITS; ++k) w[k] = packed[(size_t)t * BITS + k];
    for (int k = 0; k < 32; ++k) out[(size_t)t * 32 + k] = (int32_t)code_at_rt<BITS>(w, k);
}
template <int BITS>
__global__ __launch_bounds__(256) void k_unpack_z(const uint32_t *__restrict__ zpacked, int32_t *__restrict__ out,
                                                  uint32_t O, uint32_t G, uint32_t row_words)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= O * G) return;
    const uint32_t row = t / G, j = t - row * G;
    const uint32_t bit = j * BITS, wi = bit >> 5, sh = bit & 31u;
    uint64_t two = zpacked[row * row_words + wi];
    if (sh + BITS > 32u) two |= (uint64_t)zpacked[row * row_words + wi + 1] << 32;
    out[t] = (int32_t)((uint32_t)(two >> sh) & ((1u << BITS) - 1u));
}

// Test aid: one thread per 32-code segment of the working layout; the first n_groups threads also split the
// (s, zero point) pairs.
template <int BITS>
__global__ __launch_bounds__(256) void k_unpack_work(const uint32_t *__restrict__ work, const uint32_t *__restrict__ clampbits,
                                                     const floatx2 *__restrict__ sz, int32_t *__restrict__ codes,
                                                     uint8_t *__restrict__ clamped, float *__restrict__ zbar, uint32_t n_segs,
                                                     uint32_t n_groups)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (zbar != nullptr && t < n_groups) zbar[t] = sz[t][1];
    if (t >= n_segs) return;
    typedef WorkCodes<BITS> WC;
    if (codes != nullptr) {
        uint32_t w[WC::kWords];
#pragma unroll
        for (int k = 0; k < WC::kWords; ++k) w[k] = work[(size_t)t * WC::kWords + k];
#pragma unroll
        for (int e = 0; e < 32; ++e)
            codes[(size_t)t * 32 + e] = (int32_t)((w[WC::word_of(e)] >> WC::bit_of(e)) & ((1u << BITS) - 1u));
    }
    if (clamped != nullptr) {
        const uint32_t bits = clampbits[t];                 // bit e of the segment's word: weight e was clamped
        for (int e = 0; e < 32; ++e) clamped[(size_t)t * 32 + e] = (uint8_t)((bits >> e) & 1u);
    }
}

// ---------------------------------------------------------------------------------------------
// min/max initialisation: one lane reduces a piece of 16 bytes, a butterfly over lanes the pieces of a group.
template <typename WT> constexpr int kMinmaxPieces = sizeof(WT) == 4 ? 8 : 4;      // pieces per lane: 64 / 128 bytes in flight
struct InitBatch {
    const void *W[kMaxBatch]; float *s[kMaxBatch], *z[kMaxBatch];
    uint32_t n[kMaxBatch];                 // pieces of 16 bytes (small kernel) / groups (wave kernel)
    uint32_t g[kMaxBatch];                 // group size (wave kernel)
    uint32_t first[kMaxBatch + 1];
};

__device__ __forceinline__ void minmax_to_sz(float lo, float hi, float qmax, float *s, float *z)
{
    float step = (hi - lo) / qmax;
    if (!(step >= 1e-10f)) step = 1e-10f;
    const float zf = __builtin_rintf((-lo) / step);
    *s = step;
    *z = __builtin_fminf(__builtin_fmaxf(zf, 0.0f), qmax);
}

// One step of a butterfly over the lanes of a row, for four minima and maxima at a time: one instruction each (through LDS two and a
// wait).  Two wait states lie between the write of a register and its read by another lane.
#define EQAT_MINMAX_DPP(CTRL)                                                                                                     \
    asm("s_nop 1\n\tv_min_f32_dpp %0, %0, %0 " CTRL "\n\tv_max_f32_dpp %4, %4, %4 " CTRL "\n\tv_min_f32_dpp %1, %1, %1 " CTRL          \
        "\n\tv_max_f32_dpp %5, %5, %5 " CTRL "\n\tv_min_f32_dpp %2, %2, %2 " CTRL "\n\tv_max_f32_dpp %6, %6, %6 " CTRL                \
        "\n\tv_min_f32_dpp %3, %3, %3 " CTRL "\n\tv_max_f32_dpp %7, %7, %7 " CTRL                                                    \
        : "+v"(lo[0]), "+v"(lo[1]), "+v"(lo[2]), "+v"(lo[3]), "+v"(hi[0]), "+v"(hi[1]), "+v"(hi[2]), "+v"(hi[3]))
// minima and maxima over LANES neighbouring lanes, in all of them
template <int U, int LANES> __device__ __forceinline__ void group_minmax(float *lo, float *hi)
{
#pragma unroll
    for (int u = 0; u < U; u += 4, lo += 4, hi += 4) {
        EQAT_MINMAX_DPP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
        EQAT_MINMAX_DPP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
        if constexpr (LANES >= 8) EQAT_MINMAX_DPP("row_half_mirror row_mask:0xf bank_mask:0xf");
        if constexpr (LANES >= 16) EQAT_MINMAX_DPP("row_mirror row_mask:0xf bank_mask:0xf");
#pragma unroll
        for (int m = 16; m < LANES; m <<= 1)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lo[k] = __builtin_fminf(lo[k], __shfl_xor(lo[k], m));
                hi[k] = __builtin_fmaxf(hi[k], __shfl_xor(hi[k], m));
            }
    }
}
#undef EQAT_MINMAX_DPP

// A lane takes pieces of 16 bytes, eight weights (bf16) or four (fp32), neighbouring lanes neighbouring pieces; a wave takes U runs of 64 pieces.
// LPG = pieces of a group.  The two divisions of a group cost as much as its reduction: the lanes of a group take a run each.
// (One group at a time through LDS, with the divisions in one lane of the group: 4096 x 4096 bf16, min/max + pack, 20.4 us, so 17.7 with the
// leaner pack; the block's seven matrices 82 -> 74 alone.  Loads past the caches gain 5 us there, and the pack that follows loses them.)
template <typename WT, int LPG>
__global__ __launch_bounds__(256) void k_init_minmax_small(const InitBatch b, float qmax)
{
    constexpr int PIECE = 16 / (int)sizeof(WT), U = kMinmaxPieces<WT>, LANES = LPG < 64 ? LPG : 64;
    const int slot = batch_slot(b.first, blockIdx.x);
    const WT *__restrict__ W = reinterpret_cast<const WT *>(b.W[slot]);
    float *__restrict__ s = b.s[slot], *__restrict__ z = b.z[slot];
    const uint32_t n = b.n[slot], lane = threadIdx.x & 63u;
    // n % LPG == 0: a group never straddles the end of the array.  The runs of a workgroup's waves take turns in memory; where a group is two runs
    // long, those of a wave follow one another.
    constexpr uint32_t STRIDE = LPG == 128 ? 64u : 256u;
    const uint32_t c0 = (blockIdx.x - b.first[slot]) * (256u * U) + (STRIDE == 64u ? (threadIdx.x >> 6) * (64u * U) + lane : threadIdx.x);
    uintx4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t c = c0 + u * STRIDE;
        v[u] = *reinterpret_cast<const uintx4 *>(W + (size_t)(c < n ? c : 0u) * PIECE);
    }
    float lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        auto get = [&](int k) { return sizeof(WT) == 4 ? __uint_as_float(v[u][k & 3]) : __uint_as_float(k & 1 ? v[u][k >> 1] & 0xFFFF0000u : v[u][k >> 1] << 16); };
        lo[u] = hi[u] = get(0);
#pragma unroll
        for (int k = 1; k < PIECE; ++k) { lo[u] = __builtin_fminf(lo[u], get(k)); hi[u] = __builtin_fmaxf(hi[u], get(k)); }
    }
    group_minmax<U, LANES>(lo, hi);
    if constexpr (LPG == 128) {
#pragma unroll
        for (int u = 0; u < U; u += 2) { lo[u] = lo[u + 1] = __builtin_fminf(lo[u], lo[u + 1]); hi[u] = hi[u + 1] = __builtin_fmaxf(hi[u], hi[u + 1]); }
    }
    // Every lane of a group has its minimum and maximum now: one of them works out the group of each run (four, 16 pieces of four runs, ...).
    constexpr int TURN = LANES < U ? LANES : U;                // runs that the lanes of a group work out at a time
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += TURN) {
        const uint32_t mine = lane & (LANES - 1u);
        float l = lo[u0], h = hi[u0];
#pragma unroll
        for (int u = 1; u < TURN; ++u) { l = mine == (uint32_t)u ? lo[u0 + u] : l; h = mine == (uint32_t)u ? hi[u0 + u] : h; }
        const uint32_t c = c0 + (u0 + mine) * STRIDE;
        if (mine < (uint32_t)TURN && c < n) minmax_to_sz(l, h, qmax, s + c / LPG, z + c / LPG);
    }
}
// Any other group size: one wavefront per group.
template <typename WT>
__global__ __launch_bounds__(256) void k_init_minmax_wave(const InitBatch b, float qmax)
{
    const int slot = batch_slot(b.first, blockIdx.x);
    const WT *__restrict__ W = reinterpret_cast<const WT *>(b.W[slot]);
    float *__restrict__ s = b.s[slot], *__restrict__ z = b.z[slot];
    const uint32_t n_groups = b.n[slot], g = b.g[slot];
    const uint32_t grp = (blockIdx.x - b.first[slot]) * 4u + (threadIdx.x >> 6);
    if (grp >= n_groups) return;
    const uint32_t lane = threadIdx.x & 63u;
    const WT *base = W + (size_t)grp * g;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    for (uint32_t c = lane; c < g / 8u; c += 64u) {
        Chunk8<WT> ch;
        ch.load(base + c * 8u);
#pragma unroll
        for (int k = 0; k < 8; ++k) { lo = __builtin_fminf(lo, ch.get(k)); hi = __builtin_fmaxf(hi, ch.get(k)); }
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        lo = __builtin_fminf(lo, __shfl_xor(lo, m));
        hi = __builtin_fmaxf(hi, __shfl_xor(hi, m));
    }
    if (lane == 0) minmax_to_sz(lo, hi, qmax, s + grp, z + grp);
}

// Groups wider than a dW tile: ds / dz of group t from its n_per consecutive per-32-column partials, in one launch
// (blockIdx.y: 0 = ds, 1 = dz).  LPG lanes share a group: each adds every LPG-th partial, an xor butterfly adds the lanes:
// a fixed order.  LPG = 4 (up to eight partials): the lanes fetch them and the sum runs partial by partial, as with one lane.  One thread per group walking its
// partials alone left the chip with a few hundred wavefronts of serial, uncoalesced loads (18 us per output at 4096 groups of 128 partials, 36 us for ds and
// dz; now 6 us for both).
// `dz` (blockIdx.y = 1) is multiplied by -s[t]: the sum of the clamped dWhat becomes the gradient of the zero point.
template <int LPG>
__global__ __launch_bounds__(256) void k_reduce_partials(const float *__restrict__ part_ds, const float *__restrict__ part_dz,
                                                         float *__restrict__ ds, float *__restrict__ dz,
                                                         const float *__restrict__ s, uint32_t n_out, uint32_t n_per)
{
    const bool is_dz = blockIdx.y != 0;
    const float *__restrict__ part = is_dz ? part_dz : part_ds;
    float *__restrict__ out = is_dz ? dz : ds;
    const uint32_t t = blockIdx.x * (256u / LPG) + threadIdx.x / LPG, l = threadIdx.x % LPG;
    if (out == nullptr || t >= n_out) return;         // LPG divides the wavefront: the lanes of a group leave together
    float acc = 0.0f;
    if constexpr (LPG == 4) {
        const float lo = l < n_per ? part[(size_t)t * n_per + l] : 0.0f, hi = l + 4 < n_per ? part[(size_t)t * n_per + l + 4] : 0.0f;
#define EQAT_QUAD_LANE(V, K) __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(V), (K) * 0x55, 0xF, 0xF, true))
        acc += EQAT_QUAD_LANE(lo, 0); acc += EQAT_QUAD_LANE(lo, 1); acc += EQAT_QUAD_LANE(lo, 2); acc += EQAT_QUAD_LANE(lo, 3);
        acc += EQAT_QUAD_LANE(hi, 0); acc += EQAT_QUAD_LANE(hi, 1); acc += EQAT_QUAD_LANE(hi, 2); acc += EQAT_QUAD_LANE(hi, 3);
#undef EQAT_QUAD_LANE
    } else {
        for (uint32_t k = l; k < n_per; k += LPG) acc += part[(size_t)t * n_per + k];
#pragma unroll
        for (int m = LPG / 2; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
    }
    if (l == 0) out[t] = is_dz ? -s[t] * acc : acc;
}

// ---------------------------------------------------------------------------------------------
// host-side launchers

static inline unsigned blocks_for(size_t n, unsigned per = 256) { return (unsigned)((n + per - 1) / per); }

static inline int pow2_shift(int64_t v)
{
    for (int k = 0; k < 31; ++k) if (((int64_t)1 << k) == v) return k;
    return -1;
}

static QuantizeArgs quantize_args(const QuantizeJob &j, int unroll)
{
    const Problem &p = j.p;
    QuantizeArgs a{};
    a.zero_words = j.zero_words; a.n_zero = j.n_zero;
    a.W = j.W; a.s = j.s; a.z = j.z; a.codes = (uint32_t *)j.codes; a.clampbits = (uint8_t *)j.clampbits; a.sz = (floatx2 *)j.sz;
    a.n_chunks = (uint32_t)((size_t)p.O * p.I / 8); a.g = (uint32_t)p.g; a.g_shift = pow2_shift(p.g);
    a.n_quant_blocks = blocks_for(a.n_chunks, 256 * unroll);
    a.zpacked = (uint32_t *)j.zpacked; a.G = (uint32_t)p.G; a.row_words = (uint32_t)((p.G * p.bits + 31) / 32);
    a.n_zwords = j.zpacked != nullptr ? (uint32_t)p.O * a.row_words : 0u;
    return a;
}

// More weights than the memory-side cache holds: the backward, which reads W again, finds nothing of it there whatever the quantize pass does.  A step of
// 1000 tokens, seven matrices of 810 MB in all: 1731 us, loaded past the caches 1708; 4096 x 11008, 90 MB, 300 tokens: 165 and 172.
constexpr size_t kQuantizeOnceBytes = (size_t)256 << 20;

template <typename WT, int BITS>
static void quantize_t(const QuantizeJob *jobs, int n, bool for_pack, hipStream_t st)
{
    QuantizeBatch b{};
    uint32_t first = 0;
    const bool large_pack = for_pack && n == 1 && sizeof(WT) == 2 && (size_t)jobs[0].p.O * jobs[0].p.I / 8 >= kPackLargeChunks;
    for (int i = 0; i < n; ++i) {
        b.a[i] = quantize_args(jobs[i], large_pack ? kPackUnrollLarge : kQuantUnroll);
        b.first[i] = first;
        first += b.a[i].n_quant_blocks + blocks_for(b.a[i].n_zwords);
    }
    for (int i = n; i <= kMaxBatch; ++i) b.first[i] = first;
    size_t w_bytes = 0;
    for (int i = 0; i < n; ++i) w_bytes += (size_t)jobs[i].p.O * jobs[i].p.I * sizeof(WT);
    const bool once = w_bytes > kQuantizeOnceBytes;
    const dim3 grid(first), block(256);
    // eqat_pack: dense stream, no clamp plane;
    // the quantize pass of the Block-AP calls: working layout, clamp plane for the backward
    if constexpr (sizeof(WT) == 2) {
        if (large_pack) { k_quantize<WT, BITS, false, false, false, kPackUnrollLarge><<<grid, block, 0, st>>>(b); return; }
    }
    if (for_pack) k_quantize<WT, BITS, false, false><<<grid, block, 0, st>>>(b);
    else if (jobs[0].clampbits != nullptr && once) k_quantize<WT, BITS, true, true, true><<<grid, block, 0, st>>>(b);
    else if (jobs[0].clampbits != nullptr) k_quantize<WT, BITS, true, true><<<grid, block, 0, st>>>(b);
    else if (once) k_quantize<WT, BITS, false, true, true><<<grid, block, 0, st>>>(b);
    else k_quantize<WT, BITS, false, true><<<grid, block, 0, st>>>(b);
}

void launch_quantize_batch(const QuantizeJob *jobs, int n, bool for_pack, hipStream_t st)
{
    const Problem &p = jobs[0].p;        // all jobs share bits, weight dtype and whether a clamp plane is written
#define EQAT_Q(WT, B) quantize_t<WT, B>(jobs, n, for_pack, st)
    if (p.w_bf16) { if (p.bits == 2) EQAT_Q(bf16_t, 2); else if (p.bits == 3) EQAT_Q(bf16_t, 3); else EQAT_Q(bf16_t, 4); }
    else          { if (p.bits == 2) EQAT_Q(float, 2);  else if (p.bits == 3) EQAT_Q(float, 3);  else EQAT_Q(float, 4); }
#undef EQAT_Q
}

void launch_quantize(const Problem &p, const void *W, const float *s, const float *z, void *codes, void *clampbits,
                     void *sz, void *zpacked, bool for_pack, uint32_t *zero_words, uint32_t n_zero, hipStream_t st)
{
    const QuantizeJob j{p, W, s, z, codes, clampbits, sz, zpacked, zero_words, n_zero};
    launch_quantize_batch(&j, 1, for_pack, st);
}

void launch_e2e_prepare(const Problem &p, const void *packed, void *work, const float *s, const void *zpacked,
                        const float *zfloat, void *sz, float *zb_out, uint32_t *zero_words, uint32_t n_zero, hipStream_t st)
{
    const uint32_t n_segs = packed != nullptr ? (uint32_t)((size_t)p.O * p.I / 32) : 0u;
    const uint32_t nb = blocks_for(n_segs), n_groups = (uint32_t)((size_t)p.O * p.G);
    const uint32_t row_words = (uint32_t)((p.G * p.bits + 31) / 32);
    const dim3 grid(nb + blocks_for(n_groups)), block(256);
#define EQAT_PREP(B) k_e2e_prepare<B><<<grid, block, 0, st>>>((const uint32_t *)packed, (uint32_t *)work, n_segs, nb, s, \
                                                             (const uint32_t *)zpacked, zfloat, (floatx2 *)sz, zb_out, \
                                                             n_groups, (uint32_t)p.G, row_words, zero_words, n_zero)
    if (p.bits == 2) EQAT_PREP(2); else if (p.bits == 3) EQAT_PREP(3); else EQAT_PREP(4);
#undef EQAT_PREP
}

void launch_unpack(const Problem &p, const void *Wpacked, const void *zpacked, int32_t *codes, int32_t *zcodes, hipStream_t st)
{
    const uint32_t row_words = (uint32_t)((p.G * p.bits + 31) / 32);
    if (codes != nullptr) {
        const uint32_t n_segs = (uint32_t)((size_t)p.O * p.I / 32);
        const dim3 grid(blocks_for(n_segs)), block(256);
        if (p.bits == 2) k_unpack_codes<2><<<grid, block, 0, st>>>((const uint32_t *)Wpacked, codes, n_segs);
        else if (p.bits == 3) k_unpack_codes<3><<<grid, block, 0, st>>>((const uint32_t *)Wpacked, codes, n_segs);
        else k_unpack_codes<4><<<grid, block, 0, st>>>((const uint32_t *)Wpacked, codes, n_segs);
    }
    if (zcodes != nullptr) {
        const size_t n = (size_t)p.O * p.G;
        const dim3 grid(blocks_for(n)), block(256);
        if (p.bits == 2) k_unpack_z<2><<<grid, block, 0, st>>>((const uint32_t *)zpacked, zcodes, (uint32_t)p.O, (uint32_t)p.G, row_words);
        else if (p.bits == 3) k_unpack_z<3><<<grid, block, 0, st>>>((const uint32_t *)zpacked, zcodes, (uint32_t)p.O, (uint32_t)p.G, row_words);
        else k_unpack_z<4><<<grid, block, 0, st>>>((const uint32_t *)zpacked, zcodes, (uint32_t)p.O, (uint32_t)p.G, row_words);
    }
}

void launch_unpack_work(const Problem &p, const void *work, const void *clampbits, const void *sz, int32_t *codes,
                        uint8_t *clamped, float *zbar, hipStream_t st)
{
    const uint32_t n_segs = (uint32_t)((size_t)p.O * p.I / 32), n_groups = (uint32_t)((size_t)p.O * p.G);    // n_groups <= n_segs
    const dim3 grid(blocks_for(n_segs)), block(256);
    const uint32_t *w = (const uint32_t *)work, *c = (const uint32_t *)clampbits;
    const floatx2 *q = (const floatx2 *)sz;
    if (p.bits == 2) k_unpack_work<2><<<grid, block, 0, st>>>(w, c, q, codes, clamped, zbar, n_segs, n_groups);
    else if (p.bits == 3) k_unpack_work<3><<<grid, block, 0, st>>>(w, c, q, codes, clamped, zbar, n_segs, n_groups);
    else k_unpack_work<4><<<grid, block, 0, st>>>(w, c, q, codes, clamped, zbar, n_segs, n_groups);
}

template <typename WT>
static void init_minmax_t(const InitJob *jobs, int n, hipStream_t st)
{
    const float qmax = (float)((1 << jobs[0].p.bits) - 1);
    // one lane per 16 bytes and a butterfly over the lanes of a group when every matrix has the same group size
    // of 32 .. 512; one wavefront per group otherwise
    int64_t g = jobs[0].p.g;
    for (int i = 1; i < n; ++i) if (jobs[i].p.g != g) g = 0;
    const bool small = g == 32 || g == 64 || g == 128 || g == 256 || g == 512;
    InitBatch b{};
    uint32_t first = 0;
    for (int i = 0; i < n; ++i) {
        const Problem &p = jobs[i].p;
        b.W[i] = jobs[i].W; b.s[i] = jobs[i].s; b.z[i] = jobs[i].z; b.g[i] = (uint32_t)p.g;
        b.n[i] = small ? (uint32_t)((size_t)p.O * p.I * sizeof(WT) / 16) : (uint32_t)((size_t)p.O * p.G);
        b.first[i] = first;
        first += small ? blocks_for(b.n[i], 256 * kMinmaxPieces<WT>) : blocks_for(b.n[i], 4);
    }
    for (int i = n; i <= kMaxBatch; ++i) b.first[i] = first;
    const dim3 grid(first), block(256);
    switch (small ? (int)g : 0) {
    case 32:  k_init_minmax_small<WT, 32 * (int)sizeof(WT) / 16><<<grid, block, 0, st>>>(b, qmax); break;
    case 64:  k_init_minmax_small<WT, 64 * (int)sizeof(WT) / 16><<<grid, block, 0, st>>>(b, qmax); break;
    case 128: k_init_minmax_small<WT, 128 * (int)sizeof(WT) / 16><<<grid, block, 0, st>>>(b, qmax); break;
    case 256: k_init_minmax_small<WT, 256 * (int)sizeof(WT) / 16><<<grid, block, 0, st>>>(b, qmax); break;
    case 512: k_init_minmax_small<WT, 512 * (int)sizeof(WT) / 16><<<grid, block, 0, st>>>(b, qmax); break;
    default:  k_init_minmax_wave<WT><<<grid, block, 0, st>>>(b, qmax);
    }
}

void launch_init_minmax_batch(const InitJob *jobs, int n, hipStream_t st)
{
    if (jobs[0].p.w_bf16) init_minmax_t<bf16_t>(jobs, n, st);
    else init_minmax_t<float>(jobs, n, st);
}

void launch_init_minmax(const Problem &p, const void *W, float *s, float *z, hipStream_t st)
{
    const InitJob j{p, W, s, z};
    launch_init_minmax_batch(&j, 1, st);
}

void launch_reduce_partials(const float *part_ds, const float *part_dz, float *ds, float *dz, const float *s, size_t n_out,
                            uint32_t n_per, hipStream_t st)
{
    const uint32_t n = (uint32_t)n_out;
    // a wavefront per group as soon as a group has more partials than half of one; few partials: several groups per wavefront, up to eight summed one
    // after another, as the tile kernel adds up a group that lies inside a tile (g = 256 does in tiles of 256, not in those of 128).  Four lanes fetch them
    // where there are few groups (dW, ds, dz, 62 tokens, 768 -> 11352, g = 256, 34056 groups, us with one lane / four: 27.3 / 25.9; 374 tokens, 3072 -> 1304
    // 19.6 / 19.1), one where there are many (515 tokens, 4032 -> 11008, g = 96, 462336 groups 113.3 / 117.2; 2000 tokens, 4032 -> 4096 74.1 / 75.4).
#define EQAT_RED(L) k_reduce_partials<L><<<dim3(blocks_for(n_out, 256 / L), 2), dim3(256), 0, st>>>(part_ds, part_dz, ds, dz, s, n, n_per)
    if (n_per > 32) EQAT_RED(64); else if (n_per > 8) EQAT_RED(16); else if (n_out < 65536) EQAT_RED(4); else EQAT_RED(1);
#undef EQAT_RED
}

}  // namespace eqat
