// E2E-QP forward for a handful of tokens (decode-time matrix-vector product, App. "Speedup with BitBLAS" of the paper
// measures this shape of work):  Y[t,o] = sum_i X[t,i] * (w_q[o,i] - z[o,j]) * s[o,j],  T <= 64.
//
// HBM-bound: every weight is read once, N/8 bytes, straight from the dense packed stream of the C ABI (no re-layout
// pass, which would triple the traffic).  One workgroup owns 16 output rows; its 4 waves split the input dimension
// and meet in LDS at the end (fixed order: deterministic).  The contraction runs on v_mfma_f32_16x16x32_bf16 with
// the WEIGHTS as the A operand (16 rows x 32 k) and the tokens as the 16 columns of B, so that one byte-permute table
// per 32-code segment (WhatTable, shared with the GEMM producer) turns codes into bf16 at about one VALU
// instruction per weight and the multiply-adds cost nothing.
//
// Order of the contraction index.  A lane holds one 32-code segment of one row and feeds 8 consecutive codes of it to each
// of 4 MFMAs.  In the dense 2-bit stream, (word >> 2 k) & 0x03030303 leaves the codes k, k + 4, k + 8, k + 12 of the word
// in the four bytes of a register, and the table turns them into two registers, the pairs (k, k + 4) and (k + 8, k + 12):
// the four first pairs are the first eight codes of the word in the order 0 4 1 5 2 6 3 7, the four second pairs the other
// eight in the same order.  MFMA does not care in which order k runs as long as both operands agree, so the token rows
// are staged in LDS with every eight values in that order (slot_code()), a permutation inside 16 bytes; k_gemv_run has
// another order beside it (kPairs).  4-bit codes come
// out of their converts in any order wanted, and the dense 3-bit stream, which has no byte alignment at all, is taken twelve
// bits at a time (spread_3bit): both keep the natural order.
#include "common.h"
#include "dense_codes.h"
#include "kernels.h"

#include <algorithm>
#include <atomic>

namespace eqat {

namespace {

struct GemvArgs {
    const bf16_t *X; const uint32_t *Wp; const float *s; const uint32_t *zp; const float *zf; bf16_t *Y;
    int T, I, O, G, g;
    uint32_t spg_magic;            // ceil(2^32 / (g/32)): group of segment sg = mulhi(sg, spg_magic), exact for sg * (g/32) < 2^32
    uint32_t w_row_bytes, z_row_words;
    uint32_t x_bytes, w_bytes, s_bytes, z_bytes;
};

constexpr int kGemvRows = 16;      // output rows per workgroup (the M of the MFMA)
constexpr int kGemvWaves = 4;      // waves per workgroup, splitting the input dimension
constexpr int kGemvMaxWaves = 8;   // ... of the run kernel when it is launched with one wave per run
constexpr int kGemvUnroll = 4;     // chunks (4 segments = 128 inputs each) in flight per wave

// General group sizes: step size and zero point fetched per 32-code segment (many small scattered loads: slow, kept for
// group sizes the run kernel below does not take).  RB = 16-row blocks per workgroup.
template <int BITS, bool FLOATZ, int RB>
__global__ __launch_bounds__(64 * kGemvWaves) void k_gemv_any(const GemvArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t *xs = reinterpret_cast<bf16_t *>(smem_raw);                       // [T][I], contraction-slot order
    float *red = reinterpret_cast<float *>(smem_raw);                        // reused after the loop: [waves][RB][16][16]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int n_segs = a.I >> 5;

    // ---- stage the token rows in slot order: one 32-input segment per thread and trip, 2-byte LDS scatter with
    //      compile-time offsets
    for (int e = tid; e < a.T * n_segs; e += 64 * kGemvWaves) {
        const int n = e / n_segs, seg = e - n * n_segs;
        const bf16_t *src = a.X + (size_t)n * a.I + seg * 32;
        bf16_t *dst = xs + (size_t)n * a.I + seg * 32;
        bf16x8 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const bf16x8 *>(src + 8 * q);
#pragma unroll
        for (int c = 0; c < 32; ++c) dst[code_slot<BITS>(c)] = v[c / 8][c % 8];
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rW = make_rsrc(a.Wp, a.w_bytes);
    const __amdgpu_buffer_rsrc_t rS = make_rsrc(a.s, a.s_bytes);
    const __amdgpu_buffer_rsrc_t rZ = make_rsrc(FLOATZ ? (const void *)a.zf : (const void *)a.zp, a.z_bytes);
    int o[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) o[rb] = (blockIdx.x * RB + rb) * kGemvRows + r;
    // The waves interleave: in trip `it` wave w takes chunks [(it * waves + w) * unroll, +unroll), so that one trip of the
    // workgroup reads waves * unroll * 128 codes = one contiguous run of every row (DRAM page locality).
    const int n_chunks = (a.I + 127) / 128;
    const int c_begin = wave * kGemvUnroll, c_end = n_chunks;
    // lanes whose column is not a token multiply token 0 again; their columns of the result are never stored
    const bf16_t *xlane = xs + (size_t)((lane & 15) < a.T ? (lane & 15) : 0) * a.I;

    floatx4 acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    for (int c0 = c_begin; c0 < c_end; c0 += kGemvUnroll * kGemvWaves) {
        CodeWords<BITS> cw[kGemvUnroll][RB];
        float sv[kGemvUnroll][RB], zv[kGemvUnroll][RB];
        uint32_t zw0[kGemvUnroll][RB], zw1[kGemvUnroll][RB];
        // all loads of the unrolled chunks first
#pragma unroll
        for (int u = 0; u < kGemvUnroll; ++u) {
            const int seg = (c0 + u) * 4 + kq;
            const uint32_t j = a.spg_magic ? __umulhi((uint32_t)seg, a.spg_magic) : (uint32_t)seg;      // 0: one segment per group
            const bool seg_ok = (c0 + u) < c_end && seg < n_segs;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const bool ok = seg_ok && o[rb] < a.O;
                cw[u][rb] = load_code_words<BITS>(rW, ok ? (uint32_t)o[rb] * a.w_row_bytes + (uint32_t)seg * (4u * BITS) : kOobOffset);
                sv[u][rb] = __int_as_float(buf_load4(rS, ok ? ((uint32_t)o[rb] * (uint32_t)a.G + j) * 4u : kOobOffset));
                if constexpr (FLOATZ) {
                    zv[u][rb] = __int_as_float(buf_load4(rZ, ok ? ((uint32_t)o[rb] * (uint32_t)a.G + j) * 4u : kOobOffset));
                } else {
                    const uint32_t wi = (j * BITS) >> 5;
                    zw0[u][rb] = (uint32_t)buf_load4(rZ, ok ? ((uint32_t)o[rb] * a.z_row_words + wi) * 4u : kOobOffset);
                    zw1[u][rb] = (BITS == 3) ? (uint32_t)buf_load4(rZ, ok ? ((uint32_t)o[rb] * a.z_row_words + wi + 1u) * 4u : kOobOffset) : 0u;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kGemvUnroll; ++u) {
            const int seg = (c0 + u) * 4 + kq;
            // token fragments: lane (n, kq) holds slots kq*8.. of MFMA t of segment seg.  A segment past the end of the row
            // (or of this wave's range) has s = 0, i.e. all-zero weights: any finite token data will do for it.
            const bf16_t *xrow = xlane + (seg < n_segs ? seg : 0) * 32;
            const bf16x8 b0 = *reinterpret_cast<const bf16x8 *>(xrow + 0);
            const bf16x8 b1 = *reinterpret_cast<const bf16x8 *>(xrow + 8);
            const bf16x8 b2 = *reinterpret_cast<const bf16x8 *>(xrow + 16);
            const bf16x8 b3 = *reinterpret_cast<const bf16x8 *>(xrow + 24);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if constexpr (!FLOATZ) {
                    const uint32_t j = a.spg_magic ? __umulhi((uint32_t)seg, a.spg_magic) : (uint32_t)seg, sh = (j * BITS) & 31u;
                    const uint64_t two = (uint64_t)zw0[u][rb] | ((uint64_t)zw1[u][rb] << 32);
                    zv[u][rb] = (float)((uint32_t)(two >> sh) & ((1u << BITS) - 1u));
                }
                WhatTable<BITS> tab;
                tab.build(sv[u][rb], zv[u][rb]);
                acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(eight_of<BITS, 0>(tab, cw[u][rb]), b0, acc[rb], 0, 0, 0);
                acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(eight_of<BITS, 1>(tab, cw[u][rb]), b1, acc[rb], 0, 0, 0);
                acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(eight_of<BITS, 2>(tab, cw[u][rb]), b2, acc[rb], 0, 0, 0);
                acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(eight_of<BITS, 3>(tab, cw[u][rb]), b3, acc[rb], 0, 0, 0);
            }
        }
    }

    // ---- sum the four waves' partial tiles (wave order) and store ------------------------------------------
    __syncthreads();                                  // everyone is done reading xs
    // acc[i] = D[row 4*(lane/16) + i][col lane%16]: row = output row of the block, col = token
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[((wave * RB + rb) * 16 + 4 * kq + i) * 16 + r] = acc[rb][i];
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = tid >> 4, n = tid & 15;       // 256 threads = 16 rows x 16 tokens
        const int oo = (blockIdx.x * RB + rb) * kGemvRows + row;
        if (n < a.T && oo < a.O) {
            float v = 0.0f;
#pragma unroll
            for (int w = 0; w < kGemvWaves; ++w) v += red[((w * RB + rb) * 16 + row) * 16 + n];
            a.Y[(size_t)n * a.O + oo] = (bf16_t)v;
        }
    }
}

// The fast path.  A lane owns a RUN of 8 consecutive segments (256 inputs) of its row per trip: 16-byte loads of the
// codes, and the run's step sizes / zero points (NG = 8, 4, 2 or 1 groups per run, i.e. g = 32, 64, 128, or any multiple
// of 256) fetched with one or two wide loads instead of one small load per segment, which is what the memory path can
// sustain: per-segment 4-byte loads from 16 rows x 3 arrays thrash the 16 KB L1 and move ~7 bytes per useful byte.
// The value table is rebuilt only when the group changes.
// MW ("more waves"): launched with one wave per run of a row, 5 to 8 of them, instead of four waves that take turns.  For
// matrices with few row blocks (less than 16 waves per compute unit with four) that puts every load of the launch in
// flight at once (measured 4-7 % faster at 5120 x 5120, 13824 x 5120 and 8192 x 8192); with many row blocks the chip is
// full anyway and the fixed-size version, whose loops the compiler knows, is the faster one.
// FORM.  kFree: left to itself the compiler runs ahead over the eight segments of a run, spreading codes and converting weights
// long before their MFMAs: the quicker order for small matrices, but the more registers and the waves drift further apart, so
// that half-read lines of codes leave the L2.  kSegments: one segment after the other.  kPairs (2 bit): another slot order, in
// which a MFMA consumes both halves of what its own two lookups give; no eight weights live across a MFMA and 60 registers in
// the place of 80, eight waves per SIMD, but the token rows take a 2-byte scatter that collides on the LDS banks (with more
// than one token 3 to 30 % slower).  See run_form().
enum RunForm { kFree, kSegments, kPairs };
template <int BITS, int FORM> __host__ __device__ constexpr int run_code_slot(int c)
{
    if (FORM != kPairs) return code_slot<BITS>(c);
    const int wd = c / 16, k = c % 16, p = k % 4, q = k / 4;        // 2 bit: codes 4 q + p of a word come out of shift 2 p
    return 8 * (2 * wd + p / 2) + 4 * (p % 2) + q;
}
template <int BITS, int FORM, int T4, int NG>
__device__ __forceinline__ bf16x8 run_eight_of(const WhatTable<BITS> &tab, const CodeWords<BITS> &c)
{
    // 4 bit, us, a conversion per code / two at a time: one token, g = 32, 4096 x 11008 12.8 / 12.1, g = 64 11.9 / 11.4; g = 128 5.46 / 5.60 (4096 x 4096)
    if constexpr (FORM != kPairs) return eight_of<BITS, T4, NG >= 4 ? kTwoCodes : kWords>(tab, c);
    const uint32_t w = c.w[T4 / 2];
    uintx4 u;
    uint32_t d0, d1;
    tab.four((w >> (4 * (T4 % 2))) & 0x03030303u, d0, d1); u[0] = d0; u[1] = d1;
    tab.four((w >> (4 * (T4 % 2) + 2)) & 0x03030303u, d0, d1); u[2] = d0; u[3] = d1;
    return __builtin_bit_cast(bf16x8, u);
}

template <int BITS, bool FLOATZ, int NG, bool MW, int FORM>
__global__ __launch_bounds__(64 * (MW ? kGemvMaxWaves : kGemvWaves)) void k_gemv_run(const GemvArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t *xs = reinterpret_cast<bf16_t *>(smem_raw);                       // [T][I], contraction-slot order
    float *red = reinterpret_cast<float *>(smem_raw);                        // reused after the loop: [waves][16][16]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_waves = MW ? (int)(blockDim.x >> 6) : kGemvWaves;
    const int r = lane & 15, kq = lane >> 4;
    const int n_segs = a.I >> 5;
    const int o = blockIdx.x * kGemvRows + r;
    const bool row_ok = o < a.O;

    const __amdgpu_buffer_rsrc_t rW = make_rsrc(a.Wp, a.w_bytes);
    const __amdgpu_buffer_rsrc_t rS = make_rsrc(a.s, a.s_bytes);
    const __amdgpu_buffer_rsrc_t rZ = make_rsrc(FLOATZ ? (const void *)a.zf : (const void *)a.zp, a.z_bytes);
    constexpr int CW = 2 * BITS;                      // 16-byte loads per run of 8 segments
    constexpr int SW = NG >= 4 ? NG / 4 : 1;          // 16-byte loads of step sizes (shorter loads for NG = 2, 1)

    auto load_run = [&](int sc, uintx4 (&cq)[CW], floatx4 (&sq)[SW], floatx4 (&zq)[SW], uint32_t (&zw)[2]) {
        const int seg0 = sc * 32 + kq * 8;
        const bool ok = row_ok && seg0 < n_segs;
        const uint32_t base = (uint32_t)o * a.w_row_bytes + (uint32_t)seg0 * (4u * BITS);
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            const intx4 v = buf_load16(rW, ok ? base + 16u * q : kOobOffset);
            cq[q] = uintx4{(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
        }
        // first group of the run: runs are 256 inputs, groups NG per run (NG > 1) or a whole number of runs per group
        const uint32_t j0 = NG > 1 ? (uint32_t)(seg0 >> 3) * NG : (a.spg_magic ? __umulhi((uint32_t)seg0, a.spg_magic) : (uint32_t)seg0);
        const uint32_t gi = ok ? ((uint32_t)o * (uint32_t)a.G + j0) * 4u : kOobOffset;
        auto wide = [&](__amdgpu_buffer_rsrc_t rr, floatx4 (&dst)[SW]) {
            if constexpr (NG >= 4) {
#pragma unroll
                for (int q = 0; q < SW; ++q) {
                    const intx4 v = buf_load16(rr, ok ? gi + 16u * q : kOobOffset);
                    dst[q] = floatx4{__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3])};
                }
            } else if constexpr (NG == 2) {
                const intx2 v = buf_load8(rr, gi);
                dst[0] = floatx4{__int_as_float(v[0]), __int_as_float(v[1]), 0.0f, 0.0f};
            } else {
                dst[0] = floatx4{__int_as_float(buf_load4(rr, gi)), 0.0f, 0.0f, 0.0f};
            }
        };
        wide(rS, sq);
        if constexpr (FLOATZ) {
            wide(rZ, zq);
        } else {
            const uint32_t wi = (j0 * BITS) >> 5;
            zw[0] = (uint32_t)buf_load4(rZ, ok ? ((uint32_t)o * a.z_row_words + wi) * 4u : kOobOffset);
            zw[1] = (BITS == 3) ? (uint32_t)buf_load4(rZ, ok ? ((uint32_t)o * a.z_row_words + wi + 1u) * 4u : kOobOffset) : 0u;
        }
    };

    const int n_runs = (n_segs + 31) / 32;            // trips of one wave cover 32 segments (4 lane groups x 8)

    // ---- stage the token rows in slot order (one 32-input segment per thread and trip) ---------------------
    for (int e = tid; e < a.T * n_segs; e += 64 * n_waves) {
        const int n = e / n_segs, seg = e - n * n_segs;
        const bf16_t *src = a.X + (size_t)n * a.I + seg * 32;
        bf16_t *dst = xs + (size_t)n * a.I + seg * 32;
        bf16x8 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const bf16x8 *>(src + 8 * q);
#pragma unroll
        for (int c = 0; c < 32; ++c) dst[run_code_slot<BITS, FORM>(c)] = v[c / 8][c % 8];
    }
    __syncthreads();

    const bf16_t *xlane = xs + (size_t)((lane & 15) < a.T ? (lane & 15) : 0) * a.I;
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int sc = wave; sc < n_runs; sc += n_waves) {
        const int seg0 = sc * 32 + kq * 8;
        uintx4 cq[CW];
        floatx4 sq[SW], zq[SW];
        uint32_t zw[2] = {0u, 0u};
        load_run(sc, cq, sq, zq, zw);
        WhatTable<BITS> tab;
        const uint32_t j0 = NG > 1 ? (uint32_t)(seg0 >> 3) * NG : (a.spg_magic ? __umulhi((uint32_t)seg0, a.spg_magic) : (uint32_t)seg0);
        const uint64_t zbits = ((uint64_t)zw[0] | ((uint64_t)zw[1] << 32)) >> ((j0 * BITS) & 31u);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            constexpr int kSegsPerGroup = 8 / NG;
            const bool seg_ok = seg0 + u < n_segs;
            if (u % kSegsPerGroup == 0) {
                const int gsel = u / kSegsPerGroup;                                   // compile time after unrolling
                const float sv = sq[gsel / 4][gsel % 4];
                float zv;
                if constexpr (FLOATZ) zv = seg_ok ? zq[gsel / 4][gsel % 4] : 0.0f;
                else zv = (float)((uint32_t)(zbits >> (gsel * BITS)) & ((1u << BITS) - 1u));
                // a segment past the end of the row shares its loads with the next row: its weights are forced to zero, by
                // the step size and, as a float zero point may be infinite or NaN there, by that too
                tab.build(seg_ok ? sv : 0.0f, zv);
            }
            CodeWords<BITS> cw;
#pragma unroll
            for (int k = 0; k < BITS; ++k) cw.w[k] = cq[(u * BITS + k) / 4][(u * BITS + k) % 4];
            const bf16_t *xrow = xlane + (seg_ok ? seg0 + u : 0) * 32;
            const bf16x8 b0 = *reinterpret_cast<const bf16x8 *>(xrow + 0);
            const bf16x8 b1 = *reinterpret_cast<const bf16x8 *>(xrow + 8);
            const bf16x8 b2 = *reinterpret_cast<const bf16x8 *>(xrow + 16);
            const bf16x8 b3 = *reinterpret_cast<const bf16x8 *>(xrow + 24);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(run_eight_of<BITS, FORM, 0, NG>(tab, cw), b0, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(run_eight_of<BITS, FORM, 1, NG>(tab, cw), b1, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(run_eight_of<BITS, FORM, 2, NG>(tab, cw), b2, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(run_eight_of<BITS, FORM, 3, NG>(tab, cw), b3, acc, 0, 0, 0);
            if constexpr (FORM == kSegments) __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- sum the waves' partial tiles (wave order) and store ------------------------------------------
    __syncthreads();                                  // everyone is done reading xs
#pragma unroll
    for (int i = 0; i < 4; ++i) red[(wave * 16 + 4 * kq + i) * 16 + r] = acc[i];
    __syncthreads();
    if (!MW || tid < 256) {
        const int row = tid >> 4, n = tid & 15;       // 256 threads = 16 rows x 16 tokens
        const int oo = blockIdx.x * kGemvRows + row;
        if (n < a.T && oo < a.O) {
            float v = 0.0f;
#pragma unroll 4
            for (int w = 0; w < n_waves; ++w) v += red[(w * 16 + row) * 16 + n];
            a.Y[(size_t)n * a.O + oo] = (bf16_t)v;
        }
    }
}

// More tokens (up to 64) than the kernels above stage at once.  The tokens a wave needs are those of its own run only, so
// nothing is shared between the waves of a workgroup: each streams its piece of the token rows through a small patch of
// LDS of its own, SUB segments of every lane group at a time, with the next piece already
// on its way into registers, and the main loop has no barrier.  Runs are half as long as above (RS = 4 segments, 512 inputs per wave and trip): the waves
// of a long row spread more evenly, and the tokens weigh more per run.  LDS rows are 16 bytes longer than
// their data (the 8 lanes served together read 8 rows) and the four 16-byte chunks of a segment are XOR-permuted with the
// lane group.
// What bounds it: up to 16 tokens the loads of codes in flight (as above); beyond that the tokens, which every workgroup
// of RB 16-row blocks reads out of L2 once.  Neighbouring lanes fetch neighbouring 16-byte chunks (a segment per lane, 64
// bytes apart, ran at 16 bytes per clock and compute unit: 11008 x 4096, 64 tokens 57 -> 37 us), and two row blocks share
// the tokens when that still leaves a workgroup for every compute unit (O >= 8192; 64 tokens, 28672 x 8192: 138 -> 96 us,
// 8192 x 28672: 130 -> 80 us; with fewer rows one block is faster: 4096 x 11008 17 instead of 23 us at 24 tokens).
// Measured against what these sizes took before (codes re-laid, then a 128 x 128-tile GEMM on a few compute units):
// 8 tokens, 3 bit: 13824 x 5120 68 -> 16 us; 8 tokens, 4 bit: 4096 x 11008 127 -> 14 us; 32 tokens, 2 bit: 4096 x 4096
// 46 -> 10 us, 28672 x 8192 109 -> 52 us; 64 tokens, 2 bit: 4096 x 4096 46 -> 16 us, 28672 x 8192 110 -> 96 us.
// Groups of 32 with two row blocks (four step sizes and zero points per run and block) spill 100 to 180 bytes a lane and are
// the slower for it, but not slower than what they replace: 32 tokens, 28672 x 8192, 2 bit: g = 128 105 -> 53 us, g = 32
// 128 -> 89; 8192 x 8192, 4 bit: 96 -> 21, 100 -> 34.
constexpr int kWideRS = 4;              // segments per lane and run
template <int TR, bool DIRECT> constexpr int kWideSub = TR >= 64 ? 1 : TR >= 16 || DIRECT ? 2 : 4;              // TR: token rows of the patch
template <int TR, bool DIRECT> constexpr int kWideRowBytes = 4 * kWideSub<TR, DIRECT> * 64 + 16;
// What a wave fetches of the weights per run and 16-row block, straight into LDS: row pieces of 16 segments of codes, then the step sizes and
// zero points of their groups.  The chunk c (16 bytes) of a row lies where the 16 rows that a read serves together meet different banks.
template <int BITS, int SRC, int NG> struct WideRun {
    static constexpr int WPS = SRC == kWorking ? WorkCodes<BITS>::kWords : BITS;                  // words per segment (the working layout is read by the lanes)
    static constexpr int CPR = 4 * WPS;                                                           // chunks of a row piece
    static constexpr int CODES = 16 * CPR * 16, S = NG * 256, Z = SRC == kPackedZ ? 256 : NG * 256, BYTES = CODES + S + Z;
    static __device__ __forceinline__ int place(int row, int c)
    {
        if constexpr (CPR == 8) return c ^ ((row >> 1) & 7);
        else if constexpr (CPR == 16) return c ^ (row & 15);
        else { const int t = c + 3 * ((row >> 2) & 3); return t >= 12 ? t - 12 : t; }             // a lane's three chunks stay side by side
    }
    static __device__ __forceinline__ int chunk_at(int row, int at)                               // the chunk that lies there
    {
        if constexpr (CPR != 12) return place(row, at);
        else { const int t = at - 3 * ((row >> 2) & 3); return t < 0 ? t + 12 : t; }
    }
};
// Where a wave fetches them so, and the next run's under the arithmetic of this one's last piece: up to 8 tokens.  The lanes
// that use them read 8 to 16 bytes of 16 rows x 4 places per instruction otherwise, every line several times: with many waves in flight it has left the
// first cache in between (such loads marked non-temporal cost 10-25 %).  What decides beside that, with many row blocks, is how many waves the LDS leaves room for: a patch
// of two segments a lane group, 8 KB a wave in all.  us, by the lanes / so: 8 tokens, 3 bit, 5120 / 13824 block 98 / 86 (with a patch of four segments 102, of one 92),
// 2 bit, 28672 x 8192 29.4 / 26.6.  More tokens leave no such room: 16 tokens, 2 bit, 4096 / 11008 50 / 55, 13 tokens, 3 bit, 3200 /
// 10880 54 / 60 (though 5120 / 13824 118 / 111), 24 tokens, 3 bit, g = 32 88 / 90.
template <int SRC, int TR> constexpr bool kWideDirect = SRC != kWorking && TR == 8;
template <int BITS, int SRC, int NG, int TR, int RB, bool DIRECT>
constexpr int kWideWaveBytes = TR * kWideRowBytes<TR, DIRECT> + (DIRECT ? RB * WideRun<BITS, SRC, NG>::BYTES : 0);
// Where the pieces are the faster way.  A wave with little to fetch ahead waits the longer for its first run: 1024 inputs, 0.2 to 0.5 us of 3 to 4.  8 tokens, us, by the
// lanes (the whole run's tokens in the patch, 2-bit codes a run ahead in registers) / so, over 1024 to 28672 inputs and 256 to 28672 rows:
// - 2 bit, and 3 bit with packed zero points: from 2048 inputs on (four runs).  2 bit, g = 128: 1024 -> 1024 3.02 / 3.23, 2048 -> 1024 3.53 / 3.42, 4096 -> 4096 4.90 / 4.60, 4096 -> 11008
//   10.1 / 8.5; 3 bit 2048 -> 1024 4.17 / 3.76, 8192 -> 4096 9.1 / 7.7, 28672 -> 1024 21.0 / 16.9.  (Rows that end just behind a run in few rows: 2816 -> 352 3.79 / 3.91.)
// - groups of 32, whose four step sizes and zero points a lane reads one by one (2 bit with float z, two loads of 16 bytes by the lanes, as above): from 4096 inputs and 8192 rows on.
//   2 bit: 1024 -> 256 3.01 / 3.46, 5120 -> 256 5.40 / 5.80, 4096 -> 11008 11.1 / 10.1; 3 bit 3072 -> 11008 11.6 / 11.6, 11008 -> 1024 9.2 / 9.8, 8192 -> 28672 46.6 / 43.0.
// - 3 bit, float z: from 4096 inputs and 8192 rows on, or 8192 inputs.  1024 -> 4096 3.75 / 3.82, 2048 -> 4096 4.16 / 4.29, 3072 -> 11008 9.8 / 9.9, 4096 -> 11008 11.3 / 10.9, 8192 -> 4096 9.0 / 8.0.
// - 4 bit, 16 bytes a lane and segment, as wide as the pieces: from 8192 inputs and more than 2^26 weights on.  28672 x 8192, the longer side the inputs 42.6 / 36.8, the rows
//   41.1 / 39.1; 13824 -> 5120 17.8 / 16.4; 11008 -> 4096 9.0 / 9.8, 8192 -> 8192, one group per row 12.1 / 13.0, 5120 -> 13824 13.8 / 14.5.
static bool wide_pieces_gain(int bits, int groups, bool floatz, int I, int O)
{
    if (bits == 4) return I >= 8192 && (int64_t)I * O > (int64_t)1 << 26;
    const bool few_words = groups < 4;
    if (bits == 2 ? few_words || floatz : few_words && !floatz) return I >= 2048;
    return (I >= 4096 && O >= 8192) || (few_words && I >= 8192);
}

// KEEP: masked 4-bit words stay words, see wide_keeps_words below (then two codes are converted at a time, but for groups of 32 in the largest form, which has no
// registers for it: 24 tokens, 7168 x 12288 45 us, 48 in pairs)
template <int BITS, int SRC, int NG, int TR, int RB, bool KEEP, bool DIRECT>
__global__ __launch_bounds__(64 * kGemvMaxWaves) void k_gemv_wide(const GemvArgs a)
{
    typedef WideRun<BITS, SRC, NG> L;
    constexpr int RS = kWideRS, SUB = kWideSub<TR, DIRECT>, ROWB = kWideRowBytes<TR, DIRECT>, NB = (TR + 15) / 16, WPS = L::WPS, XC = TR * SUB / 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_waves = (int)(blockDim.x >> 6);
    const int r = lane & 15, kq = lane >> 4;
    const int n_segs = a.I >> 5, n_runs = (n_segs + 4 * RS - 1) / (4 * RS);
    const int o0 = blockIdx.x * (RB * kGemvRows), my0 = o0 + r;              // first row of block 0, this lane's
    unsigned char *const patch = smem_raw + wave * kWideWaveBytes<BITS, SRC, NG, TR, RB, DIRECT>;
    unsigned char *const stage = patch + TR * ROWB;

    const __amdgpu_buffer_rsrc_t rX = make_rsrc(a.X, a.x_bytes);
    const RawRsrc rW = make_raw_rsrc(a.Wp, a.w_bytes), rS = make_raw_rsrc(a.s, a.s_bytes);
    const RawRsrc rZ = make_raw_rsrc(SRC == kFloatZ ? (const void *)a.zf : (const void *)a.zp, a.z_bytes);

    // Piece `sub` of run `sc`: 16-byte chunk i of this lane is number (lane + 64 i) of [token][lane group][SUB][4], so that
    // neighbouring lanes read neighbouring chunks; tokens and segments past the end come as zeros.
    uintx4 xr[XC];
    auto fetch_tokens = [&](int sc, int sub) {
#pragma unroll
        for (int i = 0; i < XC; ++i) {
            const int e = lane + 64 * i, n = e / (16 * SUB), part = (e / 4) % (4 * SUB);
            const int seg = (sc * 4 + part / SUB) * RS + sub * SUB + part % SUB;
            const uint32_t off = (n < a.T && seg < n_segs) ? ((uint32_t)n * (uint32_t)a.I + (uint32_t)(seg * 32 + (e % 4) * 8)) * 2u : kOobOffset;
            const intx4 v = buf_load16(rX, off);
            xr[i] = uintx4{(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
        }
    };
    auto stage_tokens = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();              // LDS accesses of a wave complete in order
#pragma unroll
        for (int i = 0; i < XC; ++i) {
            const int e = lane + 64 * i, n = e / (16 * SUB), part = (e / 4) % (4 * SUB);
            *reinterpret_cast<bf16x8 *>(patch + n * ROWB + part * 64 + (((e % 4) ^ (part / SUB)) * 16)) = slots_of<BITS>(__builtin_bit_cast(bf16x8, xr[i]));
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    };

    floatx4 acc[RB][NB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[rb][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    auto group_of = [&](int seg) { return NG > 1 ? (uint32_t)(seg / RS) * NG : __umulhi((uint32_t)seg, a.spg_magic); };      // of a lane's first segment
    // Codes, step sizes and zero points of run `sc`.  Neighbouring lanes fetch neighbouring chunks of a row.  Rows past O are out of range (zeros); past the
    // end of a row comes what follows it: the weights there are forced to zero.
    const uint32_t stage_lds = lds_addr_of(stage);
    uint32_t coff[RB][WPS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < WPS; ++i) {
            const int e = lane + 64 * i, row = e / L::CPR, o = o0 + rb * kGemvRows + row;
            coff[rb][i] = o < a.O ? (uint32_t)o * a.w_row_bytes + (uint32_t)(L::chunk_at(row, e % L::CPR) * 16) : kOobOffset;
        }
    [[maybe_unused]] auto issue_run = [&](int sc) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const uint32_t at = stage_lds + (uint32_t)(rb * L::BYTES);
#pragma unroll
            for (int i = 0; i < WPS; ++i) load_to_lds16_at(rW, at + (uint32_t)(i * 1024), coff[rb][i] + (uint32_t)sc * (uint32_t)(L::CPR * 16));
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                const int e = lane + 64 * i, o = o0 + rb * kGemvRows + e / (4 * NG), k = e % (4 * NG);
                const uint32_t gi = (uint32_t)o * (uint32_t)a.G + (NG > 1 ? (uint32_t)(sc * 4 * NG + k) : group_of((sc * 4 + k) * RS));
                const bool ok = o < a.O;
                load_to_lds4_at(rS, at + (uint32_t)(L::CODES + i * 256), ok ? gi * 4u : kOobOffset);
                if constexpr (SRC == kFloatZ) load_to_lds4_at(rZ, at + (uint32_t)(L::CODES + L::S + i * 256), ok ? gi * 4u : kOobOffset);
            }
            if constexpr (SRC == kPackedZ) {          // four words of a row hold the zero points of a run wherever they begin
                const int o = o0 + rb * kGemvRows + (lane >> 2);
                const uint32_t w0 = (group_of(sc * 4 * RS) * BITS) >> 5;
                load_to_lds4_at(rZ, at + (uint32_t)(L::CODES + L::S), o < a.O ? ((uint32_t)o * a.z_row_words + w0 + (uint32_t)(lane & 3)) * 4u : kOobOffset);
            }
        }
    };
    struct Run { uintx4 cq[RB][WPS]; float sq[RB][NG], zq[RB][NG]; uint32_t zw[RB][2]; };
    // the same by the lanes that use them
    [[maybe_unused]] const __amdgpu_buffer_rsrc_t bW = make_rsrc(a.Wp, a.w_bytes), bS = make_rsrc(a.s, a.s_bytes), bZ = make_rsrc(SRC == kFloatZ ? (const void *)a.zf : (const void *)a.zp, a.z_bytes);
    auto fetch_run = [&](int sc, Run &into) {
        const int seg0 = (sc * 4 + kq) * RS;
        const uint32_t j0 = group_of(seg0);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int o = my0 + rb * kGemvRows;
            const bool ok = o < a.O && seg0 < n_segs;
            const uint32_t base = (uint32_t)o * a.w_row_bytes + (uint32_t)seg0 * (4u * WPS);
#pragma unroll
            for (int q = 0; q < WPS; ++q) {
                const intx4 v = buf_load16(bW, ok ? base + 16u * q : kOobOffset);
                into.cq[rb][q] = uintx4{(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
            }
            const uint32_t gi = ok ? ((uint32_t)o * (uint32_t)a.G + j0) * 4u : kOobOffset;
            auto wide = [&](__amdgpu_buffer_rsrc_t rr, float (&dst)[NG]) {
                if constexpr (NG == 4) {
                    const intx4 v = buf_load16(rr, gi);
#pragma unroll
                    for (int k = 0; k < 4; ++k) dst[k] = __int_as_float(v[k]);
                } else if constexpr (NG == 2) {
                    const intx2 v = buf_load8(rr, gi);
                    dst[0] = __int_as_float(v[0]); dst[1] = __int_as_float(v[1]);
                } else {
                    dst[0] = __int_as_float(buf_load4(rr, gi));
                }
            };
            if constexpr (SRC == kWorking) {
#pragma unroll
                for (int k = 0; k < NG; ++k) {
                    const intx2 v = buf_load8(bS, ok ? ((uint32_t)o * (uint32_t)a.G + j0 + k) * 8u : kOobOffset);
                    into.sq[rb][k] = __int_as_float(v[0]); into.zq[rb][k] = __int_as_float(v[1]);
                }
            } else {
                wide(bS, into.sq[rb]);
            }
            if constexpr (SRC == kFloatZ) {
                wide(bZ, into.zq[rb]);
            } else if constexpr (SRC == kPackedZ) {
                const uint32_t wi = (j0 * BITS) >> 5;
                into.zw[rb][0] = (uint32_t)buf_load4(bZ, ok ? ((uint32_t)o * a.z_row_words + wi) * 4u : kOobOffset);
                into.zw[rb][1] = (BITS == 3) ? (uint32_t)buf_load4(bZ, ok ? ((uint32_t)o * a.z_row_words + wi + 1u) * 4u : kOobOffset) : 0u;
            }
        }
    };
    [[maybe_unused]] auto read_run = [&](int sc, Run &into) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const unsigned char *const at = stage + rb * L::BYTES;
#pragma unroll
            for (int q = 0; q < WPS; ++q) into.cq[rb][q] = *reinterpret_cast<const uintx4 *>(at + r * (L::CPR * 16) + L::place(r, kq * WPS + q) * 16);
            const float *const sp = reinterpret_cast<const float *>(at + L::CODES) + (r * 4 + kq) * NG, *const zp = sp + L::S / 4;
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                into.sq[rb][k] = sp[k];
                if constexpr (SRC == kFloatZ) into.zq[rb][k] = zp[k];
            }
            if constexpr (SRC == kPackedZ) {
                const uint32_t w0 = (group_of(sc * 4 * RS) * BITS) >> 5, wi = ((group_of((sc * 4 + kq) * RS) * BITS) >> 5) - w0;
                const uint32_t *const zw = reinterpret_cast<const uint32_t *>(at + L::CODES + L::S) + r * 4 + wi;
                into.zw[rb][0] = zw[0];
                into.zw[rb][1] = BITS == 3 ? zw[1] : 0u;
            }
        }
    };

    constexpr int kCodes = !KEEP ? kFields : NG == 4 && TR >= 32 && RB == 2 ? kWords : kTwoCodes;
    // By the lanes a run ahead where that costs no waves: 2-bit codes and few tokens (13824 x 5120, 8 tokens 17 -> 12 us; 4 bit or 16 tokens 5-15 % slower).
    constexpr bool AHEAD = !DIRECT && TR == 8 && BITS == 2;
    Run run;
    [[maybe_unused]] Run next;
    // Past the last run the tokens' loads are all out of range.  Leaving them out takes a branch, which the compiler moves no instruction across.  Without them: 24 tokens, 4 bit, g = 32,
    // 4096 / 11008 block 114 -> 95 us, 16 tokens, 2 bit 51 -> 48, 60 tokens, 2 bit, 8192 x 8192 27.3 -> 25.2; over 90 random sizes each, 2 bit 9 to 16 and 33 to 64 tokens 1 to 22 % faster but for a few of 2 %, 17 to
    // 32 tokens 1 to 4 % faster from 20 runs on and as much slower in short rows.  Elsewhere the branch costs as often as it gains (24 tokens, 3 bit, g = 32 88 / 90 us
    // without the loads, 4 bit, g = 64 93 / 94.5; 10 tokens, 4 bit, 1792 / 5760 34.1 / 34.9) and the loads are issued.
    constexpr bool kLastRunAsks = TR == 8 ? !DIRECT : !(BITS == 2 || (TR == 16 && BITS == 3) || (BITS == 4 && NG == 4));
    if constexpr (AHEAD) fetch_run(wave, next);
    if (wave < n_runs) {
        if constexpr (DIRECT) issue_run(wave);
        fetch_tokens(wave, 0);
    }
    for (int sc = wave; sc < n_runs; sc += n_waves) {
        const int seg0 = (sc * 4 + kq) * RS;
        const uint32_t j0 = group_of(seg0);
        if constexpr (AHEAD) { run = next; fetch_run(sc + n_waves, next); }
        else if constexpr (!DIRECT) fetch_run(sc, run);
        WhatTable<BITS> tab[RB];
#pragma unroll
        for (int sub = 0; sub < RS / SUB; ++sub) {
            stage_tokens();
            if (DIRECT && sub == 0) {
                __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));      // the run's weights were asked for before these tokens
                asm volatile("" ::: "memory");
                read_run(sc, run);
            }
            if (sub + 1 < RS / SUB) {
                fetch_tokens(sc, sub + 1);
            } else if (kLastRunAsks ? true : sc + n_waves < n_runs) {
                if constexpr (DIRECT) {
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): this run's weights have left LDS
                    asm volatile("" ::: "memory");
                    issue_run(sc + n_waves);
                }
                fetch_tokens(sc + n_waves, 0);
            }
#pragma unroll
            for (int k = 0; k < SUB; ++k) {
                const int u = sub * SUB + k;
                constexpr int kSegsPerGroup = RS / NG;
                bf16x8 w[RB][4];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    if (u % kSegsPerGroup == 0) {
                        const int gsel = u / kSegsPerGroup;
                        float zv;
                        if constexpr (SRC != kPackedZ) zv = seg0 + u < n_segs ? run.zq[rb][gsel] : 0.0f;
                        else zv = (float)((uint32_t)((((uint64_t)run.zw[rb][0] | ((uint64_t)run.zw[rb][1] << 32)) >> ((j0 * BITS) & 31u)) >> (gsel * BITS)) & ((1u << BITS) - 1u));
                        // a segment past the end of the row shares its loads with the next row: its weights are forced to zero (see k_gemv_run)
                        tab[rb].build(seg0 + u < n_segs ? run.sq[rb][gsel] : 0.0f, zv);
                    } else if (seg0 + u >= n_segs) {
                        tab[rb].build(0.0f, 0.0f);
                    }
                    if constexpr (SRC == kWorking) {
                        WorkCodes<BITS> cw;
#pragma unroll
                        for (int j = 0; j < WPS; ++j) cw.w[j] = run.cq[rb][(u * WPS + j) / 4][(u * WPS + j) % 4];
                        w[rb][0] = slots_of<BITS>(tab[rb].template eight<0>(cw)); w[rb][1] = slots_of<BITS>(tab[rb].template eight<1>(cw));
                        w[rb][2] = slots_of<BITS>(tab[rb].template eight<2>(cw)); w[rb][3] = slots_of<BITS>(tab[rb].template eight<3>(cw));
                    } else {
                        CodeWords<BITS> cw;
#pragma unroll
                        for (int j = 0; j < WPS; ++j) cw.w[j] = run.cq[rb][(u * WPS + j) / 4][(u * WPS + j) % 4];
                        w[rb][0] = eight_of<BITS, 0, kCodes>(tab[rb], cw); w[rb][1] = eight_of<BITS, 1, kCodes>(tab[rb], cw);
                        w[rb][2] = eight_of<BITS, 2, kCodes>(tab[rb], cw); w[rb][3] = eight_of<BITS, 3, kCodes>(tab[rb], cw);
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const unsigned char *const row = patch + (TR == 8 ? r & 7 : b * 16 + r) * ROWB + (kq * SUB + k) * 64;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(row + ((t ^ kq) * 16));
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) acc[rb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[rb][t], x, acc[rb][b], 0, 0, 0);
                    }
                }
            }
        }
    }

    // ---- sum the waves' partial tiles (wave order) and store: consecutive outputs of a token from consecutive lanes ----
    constexpr int ROWS = RB * kGemvRows;
    __syncthreads();
    float *const red = reinterpret_cast<float *>(smem_raw);                  // [waves][tokens][rows]
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[((wave * NB + b) * 16 + r) * ROWS + rb * kGemvRows + 4 * kq + i] = acc[rb][b][i];
    __syncthreads();
    for (int e = tid; e < a.T * ROWS; e += 64 * n_waves) {
        const int n = e / ROWS, oo = blockIdx.x * ROWS + e % ROWS;
        if (oo >= a.O) continue;
        float v = 0.0f;
        for (int w = 0; w < n_waves; ++w) v += red[(w * NB * 16 + n) * ROWS + e % ROWS];
        a.Y[(size_t)n * a.O + oo] = (bf16_t)v;
    }
}

}  // namespace

// all token rows staged in LDS at once (k_gemv_run, k_gemv_any)
static bool gemv_tokens_fit(const Problem &p) { return p.T <= 16 && (size_t)p.T * p.I * 2 <= 64 * 1024; }
// Waves per row block of k_gemv_run: one per run of 1024 inputs when four would leave the chip short of waves.
static int gemv_run_waves(const Problem &p)
{
    const int n_blocks = (int)((p.O + kGemvRows - 1) / kGemvRows), n_runs = (int)((p.I / 32 + 31) / 32);
    const bool more = n_runs > kGemvWaves && n_blocks * kGemvWaves < 16 * 256;
    return more ? std::min(n_runs, kGemvMaxWaves) : kGemvWaves;
}
// groups per run of k_gemv_wide (128 inputs of a lane); 0 = a group size it does not take
static int wide_groups(const Problem &p)
{
    if (p.g > 64 && !group_by_magic(p)) return 0;
    return p.g == 32 ? 4 : p.g == 64 ? 2 : p.g % 128 == 0 ? 1 : 0;
}

// k_gemv_wide although the tokens would fit.
// From 7 tokens on: k_gemv_run stages all token rows, 56 KB at 7 tokens of 4096 inputs, which leaves two workgroups per compute
// unit, and rows a multiple of 64 bytes apart collide on the LDS banks.  7 tokens: faster or equal at every size, width and
// group measured (one group per row: 11008 x 4096, 2 bit 15.1 -> 8.9 us, 3 bit 17.9 -> 11.6; 16384 x 2048, 4 bit 10.8 -> 8.8);
// at 5 and 6 k_gemv_run is up to 19 and 8 % the faster one (3 bit).
// Fewer tokens, 4-bit codes, more than 6144 waves (24 per compute unit; k_gemv_run<4> holds 20 to 28): a second round, and half
// read lines of codes that leave the L2 in between.  28672 x 8192, one token 71 -> 39 us, 28672 x 4096 26 -> 23.  With one
// group per run k_gemv_run needs fewer registers and has its 28 waves: one or two tokens of rows that its four waves walk in
// one trip are faster there (28672 x 4096: 20 us against 22, 40000 x 4096 27 against 30; 28672 x 4608, two trips: 24, 22).
static bool wide_is_faster(const Problem &p)
{
    if (wide_groups(p) == 0) return false;
    if (p.T >= 7) return true;
    if (p.bits != 4 || (p.O + kGemvRows - 1) / kGemvRows * gemv_run_waves(p) <= 24 * 256) return false;
    return !(p.g % 256 == 0 && p.T <= 2 && p.I > 2048 && p.I <= 4096);
}

// 17 to 64 tokens, on every forward entry point alike (bitwise equal results).  Above 32 tokens k_gemm_mid is the faster one
// where the rows fill the chip and the contraction is short.  This kernel takes about 8 us and 0.5 us per million weights
// there: 4096 x 4096 16 us against 25, 4096 x 11008 32 against 58; 13824 x 5120 40 against 30, 28672 x 8192 96 against 60.
bool gemv_work_applies(const Problem &p)
{
    if (!p.act_bf16 || wide_groups(p) == 0 || p.T <= 16 || p.T > 64) return false;
    return p.T <= 32 || 8.0 + 0.5e-6 * (double)(p.O * p.I) <= mid_us(p);
}

bool gemv_applies(const Problem &p)
{
    return p.act_bf16 && p.T >= 1 && (gemv_tokens_fit(p) || (p.T <= 16 && wide_groups(p) != 0) || gemv_work_applies(p));
}

// groups per run of k_gemv_run (256 inputs of a lane); 0 = a group size it does not take
static int run_groups(const Problem &p) { return p.g == 32 ? 8 : p.g == 64 ? 4 : p.g == 128 ? 2 : p.g % 256 == 0 ? 1 : 0; }

// Forms of k_gemv_run that exist beside the free one, and when they are taken.
// kSegments: more than 2^25 weights (the chip full of waves; fewer: up to 8 % slower, 0.3 us).  One token, free -> segment by
// segment, us: float zero points, 3 bit, g = 64 28672 x 8192 45 -> 30, 11008 x 4096 10.5 -> 9.6; 4 bit, g = 64 24000 x 8192
// 60 -> 34, g = 32 8192 x 28672 65 -> 45; 2 bit, g = 32 28672 x 8192 29.9 -> 28.0.  2 bit, g = 64 28672 x 8192 26.7 -> 23.6,
// 8192 x 8192 9.6 -> 9.3 (from 3 tokens on +-5 %, not taken).
// kPairs: 2 bit, g = 64, more waves than fit at six to a SIMD, and one token, or 8 KB of tokens, to scatter (from four tokens on
// only if all waves fit at eight: 40000 x 512, 6 tokens 8.4 us free, 9.8 in pairs).  One token: 28672 x 8192 25.5 -> 20.7
// (segment by segment 22.1), 28672 x 6144 21.0 -> 16.9 (18.6), 28672 x 4096 14.6 -> 12.0 (13.1); two: 60000 x 1024 12.5 -> 11.1
// (free); four: 28672 x 512 6.8 -> 5.7 (free).
template <int BITS, bool FLOATZ, int NG> constexpr bool kHasSegments = BITS == 2 ? NG == 4 || (FLOATZ && NG == 8) : FLOATZ && NG >= (BITS == 3 ? 2 : 4);
template <int BITS, int NG, bool MW> constexpr bool kHasPairs = BITS == 2 && NG == 4 && !MW;
static RunForm run_form(const Problem &p, bool floatz)
{
    const int ng = run_groups(p);
    const int64_t waves = (p.O + kGemvRows - 1) / kGemvRows * kGemvWaves;
    if (p.bits == 2 && ng == 4 && waves > 24 * 256 && (p.T == 1 || (p.T * p.I <= 4096 && (p.T <= 3 || waves <= 32 * 256)))) return kPairs;
    if (p.O * p.I <= (int64_t)1 << 25) return kFree;
    if (p.bits != 2) return floatz && ng >= (p.bits == 3 ? 2 : 4) ? kSegments : kFree;
    return p.T <= 2 && (ng == 4 || (floatz && ng == 8)) ? kSegments : kFree;
}

FwdRoute gemv_route(const Problem &p, bool floatz)
{
    if (gemv_tokens_fit(p) && !wide_is_faster(p)) {
        const FwdKernel kernel = run_groups(p) == 0 ? FWD_GEMV_ANY : static_cast<FwdKernel>(FWD_GEMV_RUN + run_form(p, floatz));
        return FwdRoute{kernel, 16, kGemvRows};
    }
    const int tokens = p.T <= 8 ? 8 : p.T <= 16 ? 16 : p.T <= 32 ? 32 : 64;
    return FwdRoute{FWD_GEMV_WIDE, tokens, tokens >= 32 && p.O >= 2 * kGemvRows * 256 ? 2 * kGemvRows : kGemvRows};
}

static int wide_runs(int I) { return (I / 32 + 4 * kWideRS - 1) / (4 * kWideRS); }
// 17 to 32 tokens, 4-bit codes as packed, groups of 64: with words that stay words the kernel is 2 to 15 % faster, but 2 to 6 % slower
// where all its eight waves have the same number of runs (two row blocks: one or two) or four have one each and the launch more
// than 256 workgroups.  24 tokens, us, kept / not: 4096 inputs x 4096 rows 8.3 / 7.9, 12288 x 7168 29.5 / 28.3, 2048 x 7168
// 8.4 / 8.0; 5120 x 8192 10 % the other way.  Other groups and token counts gain everywhere (8 and 12 tokens 1 to 10 %).
static bool wide_keeps_words(int I, int O, int rows)
{
    const int runs = wide_runs(I), blocks = (O + rows - 1) / rows;
    return !((runs % kGemvMaxWaves == 0 && (rows == kGemvRows || runs <= 2 * kGemvMaxWaves)) || (runs == 4 && blocks > 256));
}
template <int BITS, int SRC, int NG, int TR, int RB, bool KEEP = true, bool DIRECT = kWideDirect<SRC, TR>>
static void launch_wide_t(const GemvArgs &a, hipStream_t st)
{
    if constexpr (KEEP && BITS == 4 && SRC != kWorking && NG == 2 && TR == 32) {
        if (!wide_keeps_words(a.I, a.O, RB * kGemvRows)) return launch_wide_t<BITS, SRC, NG, TR, RB, false>(a, st);
    }
    if constexpr (DIRECT) {
        if (!wide_pieces_gain(BITS, NG, SRC == kFloatZ, a.I, a.O)) return launch_wide_t<BITS, SRC, NG, TR, RB, KEEP, false>(a, st);
    }
    auto kern = k_gemv_wide<BITS, SRC, NG, TR, RB, KEEP, DIRECT>;
    const int n_runs = wide_runs(a.I), trips = (n_runs + kGemvMaxWaves - 1) / kGemvMaxWaves;
    const int waves = (n_runs + trips - 1) / trips;
    constexpr int kWaveBytes = kWideWaveBytes<BITS, SRC, NG, TR, RB, DIRECT>;
    const size_t smem = (size_t)waves * kWaveBytes;      // at least the 1 KB per wave and token block of the final sum
    static_assert(kWaveBytes >= (TR + 15) / 16 * RB * 1024 && kGemvMaxWaves * kWaveBytes <= 160 * 1024, "LDS of the final sum, of one CU");
    // more dynamic LDS than the default limit: allowed once per instantiation and device
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kGemvMaxWaves * kWaveBytes);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    kern<<<dim3((unsigned)((a.O + RB * kGemvRows - 1) / (RB * kGemvRows))), dim3(64 * waves), smem, st>>>(a);
}
template <int BITS, int SRC>
static void launch_wide_z(int ng, const FwdRoute &way, const GemvArgs &a, hipStream_t st)
{
    const bool two = way.rows != kGemvRows;
    // the working layout comes here from 17 tokens on
#define EQAT_WIDE_NB(NG)                                                                          \
    do {                                                                                          \
        if constexpr (SRC != kWorking) {                                                          \
            if (way.tokens == 8) { launch_wide_t<BITS, SRC, NG, 8, 1>(a, st); break; }            \
            if (way.tokens == 16) { launch_wide_t<BITS, SRC, NG, 16, 1>(a, st); break; }          \
        }                                                                                         \
        if (way.tokens == 32 && !two) launch_wide_t<BITS, SRC, NG, 32, 1>(a, st);            \
        else if (way.tokens == 32) launch_wide_t<BITS, SRC, NG, 32, 2>(a, st);                    \
        else if (!two) launch_wide_t<BITS, SRC, NG, 64, 1>(a, st);                                \
        else launch_wide_t<BITS, SRC, NG, 64, 2>(a, st);                                          \
    } while (0)
    if (ng == 4) EQAT_WIDE_NB(4); else if (ng == 2) EQAT_WIDE_NB(2); else EQAT_WIDE_NB(1);
#undef EQAT_WIDE_NB
}
template <int SRC> static void launch_wide(const Problem &p, const GemvArgs &a, hipStream_t st)
{
    const int ng = wide_groups(p);
    const FwdRoute way = gemv_route(p, false);
    if (p.bits == 2) launch_wide_z<2, SRC>(ng, way, a, st);
    else if (p.bits == 3) launch_wide_z<3, SRC>(ng, way, a, st);
    else launch_wide_z<4, SRC>(ng, way, a, st);
}

static GemvArgs gemv_args(const Problem &p, const void *X, const void *codes, const void *s, void *Y)
{
    GemvArgs a{};
    a.X = (const bf16_t *)X; a.Wp = (const uint32_t *)codes; a.s = (const float *)s; a.Y = (bf16_t *)Y;
    a.T = (int)p.T; a.I = (int)p.I; a.O = (int)p.O; a.G = (int)p.G; a.g = (int)p.g;
    a.spg_magic = (p.g == 32) ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)(p.g / 32) - 1) / (uint64_t)(p.g / 32));
    a.x_bytes = (uint32_t)(p.T * p.I * 2);
    return a;
}

void launch_gemv_work(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, hipStream_t st)
{
    GemvArgs a = gemv_args(p, X, codes, sz, Y);
    a.w_row_bytes = (uint32_t)(work_code_bytes(p) / p.O);
    a.w_bytes = (uint32_t)work_code_bytes(p);
    a.s_bytes = (uint32_t)(p.O * p.G * 8);
    launch_wide<kWorking>(p, a, st);
}

void launch_gemv(const Problem &p, const void *X, const void *Wpacked, const float *s, const void *zpacked,
                 const float *zfloat, void *Y, hipStream_t st)
{
    GemvArgs a = gemv_args(p, X, Wpacked, s, Y);
    a.zp = (const uint32_t *)zpacked; a.zf = zfloat;
    a.w_row_bytes = (uint32_t)(p.I * p.bits / 8);
    a.z_row_words = (uint32_t)((p.G * p.bits + 31) / 32);
    a.w_bytes = (uint32_t)(p.O * p.I * p.bits / 8);
    a.s_bytes = (uint32_t)(p.O * p.G * 4);
    a.z_bytes = zfloat != nullptr ? a.s_bytes : (uint32_t)(p.O * a.z_row_words * 4);
    const FwdKernel kernel = gemv_route(p, zfloat != nullptr).kernel;
    if (kernel == FWD_GEMV_WIDE) {
        if (zfloat != nullptr) launch_wide<kFloatZ>(p, a, st); else launch_wide<kPackedZ>(p, a, st);
        return;
    }
    const int ng = run_groups(p);
    // a wave per run of 1024 inputs when four waves per row block would leave the chip short of waves (see k_gemv_run)
    const int n_blocks = (int)((p.O + kGemvRows - 1) / kGemvRows), waves = ng != 0 ? gemv_run_waves(p) : kGemvWaves;
    const bool more_waves = waves != kGemvWaves;
    const size_t red_bytes = (size_t)waves * 16 * 16 * 4;
    const size_t smem = (size_t)p.T * p.I * 2 > red_bytes ? (size_t)p.T * p.I * 2 : red_bytes;
    const dim3 grid((unsigned)n_blocks), block(64 * waves);
    if (ng == 1) {          // magic for "group of segment": exact for segment * (g/32) < 2^32
        a.spg_magic = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)(p.g / 32) - 1) / (uint64_t)(p.g / 32));
    }
    const RunForm form = run_form(p, zfloat != nullptr);
#define EQAT_GEMV_FORM(B, FZ, N, MW)                                                              \
    do {                                                                                          \
        if (form == kPairs) k_gemv_run<B, FZ, N, MW, kHasPairs<B, N, MW> ? kPairs : kFree><<<grid, block, smem, st>>>(a); \
        else if (form == kSegments) k_gemv_run<B, FZ, N, MW, kHasSegments<B, FZ, N> ? kSegments : kFree><<<grid, block, smem, st>>>(a); \
        else k_gemv_run<B, FZ, N, MW, kFree><<<grid, block, smem, st>>>(a);                        \
    } while (0)
#define EQAT_GEMV_NG(B, FZ, MW)                                                                   \
    do {                                                                                          \
        if (ng == 8) EQAT_GEMV_FORM(B, FZ, 8, MW);                                                  \
        else if (ng == 4) EQAT_GEMV_FORM(B, FZ, 4, MW);                                             \
        else if (ng == 2) EQAT_GEMV_FORM(B, FZ, 2, MW);                                             \
        else EQAT_GEMV_FORM(B, FZ, 1, MW);                                                          \
    } while (0)
#define EQAT_GEMV_RUN(B, FZ)                                                                      \
    do {                                                                                          \
        if (ng == 0) k_gemv_any<B, FZ, 1><<<grid, block, smem, st>>>(a);                           \
        else if (more_waves) EQAT_GEMV_NG(B, FZ, true);                                           \
        else EQAT_GEMV_NG(B, FZ, false);                                                          \
    } while (0)
#define EQAT_GEMV(B) do { if (zfloat != nullptr) EQAT_GEMV_RUN(B, true); else EQAT_GEMV_RUN(B, false); } while (0)
    if (p.bits == 2) EQAT_GEMV(2); else if (p.bits == 3) EQAT_GEMV(3); else EQAT_GEMV(4);
#undef EQAT_GEMV_RUN
#undef EQAT_GEMV_NG
#undef EQAT_GEMV_FORM
#undef EQAT_GEMV
}

}  // namespace eqat
