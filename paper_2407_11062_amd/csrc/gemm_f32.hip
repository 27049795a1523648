// fp32-activation path (parity to 1e-5): every product and sum in binary32, on v_mfma_f32_32x32x2_f32, and every
// quantisation decision from the exact binary32 quotient.
//
// The problems are small (a 512 x 512 linear at 256 tokens is 128 tiles of 32 x 32), so what bounds them is latency: the
// waves of a workgroup share one output tile and split the contraction in blocks of 32, operands come from global memory
// straight into MFMA registers without LDS or a barrier, and the waves' sums meet in LDS once, in wave order.  (Before:
// 64 x 64 tiles of scalar FMAs walked by one workgroup each, 32 of them, with an element-wise bounds check, and an epilogue of
// one thread per group: 74 + 76 + 34 + 75 us for forward, dX, dWhat and epilogue of that linear; the whole pass takes 19 now.  2048 tokens, 2048 x 2048:
// 1589 -> 655 us for all.)  The error against 64 bits halves: eight or four short chains of sums in the place of one long one.
// K order: lane half h of block k0 holds k0 + 16 h + e, e = 0 .. 15, for both operands; product e multiplies k0 + e and
// k0 + 16 + e.
#include "common.h"
#include "kernels.h"

namespace eqat {

// ---- operands: 16 consecutive contraction indices k .. k + 15 of row (or column) m; zeros outside the matrix -----------
struct RowMajorF32 {       // element (m, k) = p[m][k]
    static constexpr bool kPlain = true;
    const float *p; int rows, cols; uint32_t bytes;
    __device__ __forceinline__ void load(int m, int k, float (&v)[16]) const
    {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p, bytes);
        if (k + 16 <= cols) {
            const uint32_t off = m < rows ? ((uint32_t)m * (uint32_t)cols + (uint32_t)k) * 4u : kOobOffset;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const intx4 u = buf_load16(rs, off + 16u * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * q + e] = __int_as_float(u[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                v[e] = __int_as_float(buf_load4(rs, m < rows && k + e < cols ? ((uint32_t)m * (uint32_t)cols + (uint32_t)(k + e)) * 4u : kOobOffset));
        }
    }
};
struct ColMajorF32 {       // element (m, k) = p[k][m].  Plain loads: What of a large bf16 matrix may exceed 2 GiB here
    static constexpr bool kPlain = true;
    const float *p; int rows, cols;                      // rows: extent of k
    __device__ __forceinline__ void load(int m, int k, float (&v)[16]) const
    {
        if (m < cols && k + 16 <= rows) {
            const float *const q = p + (size_t)k * cols + m;
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = q[(size_t)e * cols];
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = m < cols && k + e < rows ? p[(size_t)(k + e) * cols + m] : 0.0f;
        }
    }
};

template <typename WT> struct FakeQuantW {   // What[o][i] from W, s, z  (Eqs.(1),(2))
    const WT *W; const float *s, *z; int O, I, g, G; float qmax;
    __device__ __forceinline__ float what(float w, float sv, float zb) const
    {
        return from_rounded(__builtin_rintf(w / sv), sv, zb);
    }
    __device__ __forceinline__ float from_rounded(float r, float sv, float zb) const
    {
        const float q = __builtin_fminf(__builtin_fmaxf(r + zb, 0.0f), qmax);
        return (q - zb) * sv;
    }
    __device__ __forceinline__ void row(int o, int i, float (&v)[16]) const     // What[o][i .. i + 15], one group
    {
        if (o >= O || i >= I) {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = 0.0f;
            return;
        }
        const size_t gi = (size_t)o * G + i / g;
        const float sv = s[gi], zb = zbar_of(z[gi], qmax);
        WT w[16];
        __builtin_memcpy(w, __builtin_assume_aligned(W + (size_t)o * I + i, 16), sizeof(w));
        // w * rcp(s) is within 2^-22 of the quotient and rounds like it unless a tie is near (or the reciprocal is no normal number):
        // only then 16 divisions, which are half of this load's arithmetic
        const float rinv = __builtin_amdgcn_rcpf(sv), as = __builtin_fabsf(sv);
        float worst = as >= 0x1p-126f && as <= 0x1p+126f ? 0.0f : 1.0f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float t = to_float(w[e]) * rinv;
            v[e] = __builtin_rintf(t);
            worst = __builtin_fmaxf(worst, __builtin_fabsf(t - v[e]));
        }
        if (worst >= 0.5f - 0x1p-20f * (zb + qmax + 2.0f)) {           // what is not clamped is below zb + qmax + 1
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = __builtin_rintf(to_float(w[e]) / sv);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = from_rounded(v[e], sv, zb);
    }
    __device__ __forceinline__ float one(int o, int i) const
    {
        const size_t gi = (size_t)o * G + i / g;
        return what(to_float(W[(size_t)o * I + i]), s[gi], zbar_of(z[gi], qmax));
    }
};

template <int BITS> struct PackedW {         // What[o][i] from packed codes and (s, z) pairs  (Eq.(2))
    const uint32_t *codes; const floatx2 *sz; int O, I, g, G;
    __device__ __forceinline__ void row(int o, int i, float (&v)[16]) const     // i a multiple of 16
    {
        if (o >= O || i >= I) {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = 0.0f;
            return;
        }
        const floatx2 p = sz[(size_t)o * G + i / g];
        const uint32_t *seg = codes + ((size_t)o * I + (i & ~31)) / 32 * BITS;
        const int h = (i >> 4) & 1;
        uint64_t bits = BITS == 2 ? seg[h] : BITS == 3 ? ((uint64_t)seg[h] | ((uint64_t)seg[h + 1] << 32)) >> (16 * h)
                                                       : (uint64_t)seg[2 * h] | ((uint64_t)seg[2 * h + 1] << 32);
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = ((float)((uint32_t)(bits >> (BITS * e)) & ((1u << BITS) - 1u)) - p[1]) * p[0];
    }
    __device__ __forceinline__ float one(int o, int i) const
    {
        const floatx2 p = sz[(size_t)o * G + i / g];
        return ((float)code_at_rt<BITS>(codes + ((size_t)o * I + (i & ~31)) / 32 * BITS, i & 31) - p[1]) * p[0];
    }
};
template <typename W> struct WeightRows {    // element (m, k) = What[m][k]
    static constexpr bool kPlain = false;
    W w;
    __device__ __forceinline__ void load(int m, int k, float (&v)[16]) const { w.row(m, k, v); }
};

// dX contracts over the rows of What: a lane would meet another (s, z) with every element, and every tile of tokens would
// divide again (2048 x 2048 x 2048: 820 us).  It reads the plain matrix that this kernel leaves in the scratch that
// dWhat takes afterwards (4 + 190 us), 16 weights per thread.
template <typename W> __device__ __forceinline__ void f32_what(const W &w, float *__restrict__ out, int64_t e)
{
    const int per_row = w.I / 16;
    if (e >= (int64_t)w.O * per_row) return;
    const int o = (int)(e / per_row), i = (int)(e - (int64_t)o * per_row) * 16;
    float v[16];
    w.row(o, i, v);
    floatx4 *const dst = reinterpret_cast<floatx4 *>(out + (size_t)o * w.I + i);
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q] = floatx4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
}
template <typename W> __global__ __launch_bounds__(256) void k_f32_what(W w, float *__restrict__ out)
{
    f32_what(w, out, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// dX of a linear with at most 32 output features: a 64 x 64 tile whose whole contraction is staged in LDS, weights rebuilt per
// tile, plain FMAs.  One launch, and token rows of O floats are read as the contiguous memory that they are; What in
// memory and MFMA tiles take a launch more and 64-byte pieces of such rows (1024 tokens, 8 x 1024: 10.2 us against 5.7).
constexpr int kShortO = 32;
template <typename W> __global__ __launch_bounds__(256) void k_f32_dx_short(const float *__restrict__ dY, W w, float *__restrict__ dX, int T)
{
    __shared__ float as[kShortO][65], bs[kShortO][65];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, tiles_n = (w.I + 63) / 64;
    const int m0 = (int)(blockIdx.x / tiles_n) * 64, n0 = (int)(blockIdx.x % tiles_n) * 64;
    for (int e = threadIdx.x; e < w.O * 64; e += 256) {
        const int m = e / w.O, k = e - m * w.O, o = e >> 6, n = e & 63;
        as[k][m] = m0 + m < T ? dY[(size_t)(m0 + m) * w.O + k] : 0.0f;
        bs[o][n] = n0 + n < w.I ? w.one(o, n0 + n) : 0.0f;
    }
    __syncthreads();
    float acc[4][4] = {};
    for (int k = 0; k < w.O; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(as[k][ty * 4 + i], bs[k][tx * 4 + j], acc[i][j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i, n = n0 + tx * 4;
        if (m < T && n < w.I) *reinterpret_cast<floatx4 *>(dX + (size_t)m * w.I + n) = floatx4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
    }
}

// C[m][n] = sum_k A(m,k) * B(n,k).  A wave's tile is 32 MB x 32 NB.  SPLIT: the NW waves of a workgroup share a tile and take
// every NW-th block of 32 of the contraction; else each has a tile of its own, side by side along M (along_m) or N.
template <int NW, bool SPLIT> struct F32Sums { float v[SPLIT ? NW : 1][32][33]; };
template <typename OpA, typename OpB, int MB, int NB, int NW, bool SPLIT>
__device__ __forceinline__ void f32_tile(const OpA &a, const OpB &b, float *__restrict__ C, int M, int N, int K, bool along_m, int bx, int by,
                                         F32Sums<NW, SPLIT> &sums)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, h = lane >> 5;
    const int m0 = (!SPLIT && along_m ? by * NW + wave : by) * (32 * MB);
    const int n0 = (!SPLIT && !along_m ? bx * NW + wave : bx) * (32 * NB);
    floatx16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    // Plain operands of a 32 x 32 tile: the next block is loaded while one is multiplied, the chain of a wave is loads that wait on
    // memory otherwise (backward: 256 x 512 x 512 14.3 -> 12.9 us, 512 x 512 x 1024 30.4 -> 23.7).  Rebuilt weights (forward 512 x 512
    // x 512: 7.9 -> 8.7) and 64 x 64 tiles (backward 2048 x 2048 x 2048: 380 -> 433) lose more by the registers than they gain.
    if constexpr (SPLIT && MB * NB == 1 && OpA::kPlain && OpB::kPlain) {
        float va[2][16], vb[2][16];
        auto load = [&](int k0, int to) {
            a.load(m0 + r, k0 + 16 * h, va[to]);
            b.load(n0 + r, k0 + 16 * h, vb[to]);
        };
        auto multiply = [&](int from) {
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[from][e], vb[from][e], acc[0][0], 0, 0, 0);
        };
        constexpr int kStep = 32 * NW;
        if (wave * 32 < K) load(wave * 32, 0);
        for (int k0 = wave * 32; k0 < K; k0 += 2 * kStep) {
            if (k0 + kStep < K) load(k0 + kStep, 1);
            multiply(0);
            if (k0 + kStep >= K) break;
            if (k0 + 2 * kStep < K) load(k0 + 2 * kStep, 0);
            multiply(1);
        }
    } else {
        for (int k0 = SPLIT ? wave * 32 : 0; k0 < K; k0 += SPLIT ? 32 * NW : 32) {
            float va[MB][16], vb[NB][16];
#pragma unroll
            for (int i = 0; i < MB; ++i) a.load(m0 + 32 * i + r, k0 + 16 * h, va[i]);
#pragma unroll
            for (int j = 0; j < NB; ++j) b.load(n0 + 32 * j + r, k0 + 16 * h, vb[j]);
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][e], vb[j][e], acc[i][j], 0, 0, 0);
        }
    }
    // acc[..][e] of a lane: row 8 (e / 4) + 4 h + e % 4, column r of the block
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = m0 + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3), n = n0 + 32 * j + r;
                    if (m < M && n < N) C[(size_t)m * N + n] = acc[i][j][e];
                }
        return;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (i + j > 0) __syncthreads();
#pragma unroll
            for (int e = 0; e < 16; ++e) sums.v[wave][8 * (e >> 2) + 4 * h + (e & 3)][r] = acc[i][j][e];
            __syncthreads();
            for (int e = threadIdx.x; e < 1024; e += 64 * NW) {
                const int m = e >> 5, n = e & 31;
                float v = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w) v += sums.v[w][m][n];
                if (m0 + 32 * i + m < M && n0 + 32 * j + n < N) C[(size_t)(m0 + 32 * i + m) * N + n0 + 32 * j + n] = v;
            }
        }
}
template <typename OpA, typename OpB, int MB, int NB, int NW, bool SPLIT>
__global__ __launch_bounds__(64 * NW) void k_f32_gemm(OpA a, OpB b, float *__restrict__ C, int M, int N, int K, bool along_m)
{
    __shared__ F32Sums<NW, SPLIT> sums;
    f32_tile<OpA, OpB, MB, NB, NW, SPLIT>(a, b, C, M, N, K, along_m, blockIdx.x, blockIdx.y, sums);
}

// Per-group epilogue of the backward: 32 lanes per group t = (o, j), consecutive in-features on consecutive lanes.
template <typename WT> struct EpilogueBlockAp {              // Eqs.(3)-(5)
    const float *dwhat; const WT *W; const float *s, *z; WT *dW; float *ds, *dz; int O, I, g, G; float qmax;
    __device__ __forceinline__ void group(int t, int lane) const
    {
        if (t >= O * G) return;
        const int o = t / G, j = t - o * G;
        const float sv = s[t], zb = zbar_of(z[t], qmax);
        float gs = 0.0f, gz = 0.0f;
        for (int i = j * g + lane; i < (j + 1) * g; i += 32) {
            const size_t e = (size_t)o * I + i;
            const float d = dwhat[e];
            const float tq = to_float(W[e]) / sv;
            const float r = __builtin_rintf(tq);
            const float qpre = r + zb;
            float cs, cw;
            if (qpre < 0.0f)       { cs = -zb;        gz += d; cw = 0.0f; }
            else if (qpre > qmax)  { cs = qmax - zb;  gz += d; cw = 0.0f; }
            else                   { cs = r - tq;              cw = 1.0f; }
            gs = __builtin_fmaf(d, cs, gs);
            if (dW != nullptr) dW[e] = (WT)(d * cw);
        }
        for (int k = 16; k >= 1; k >>= 1) { gs += __shfl_xor(gs, k, 32); gz += __shfl_xor(gz, k, 32); }
        if (lane != 0) return;
        if (ds != nullptr) ds[t] = gs;
        if (dz != nullptr) dz[t] = -sv * gz;
    }
};
template <int BITS> struct EpilogueE2e {
    const float *dwhat; const uint32_t *codes; const floatx2 *sz; float *ds, *dz; int O, I, g, G;
    __device__ __forceinline__ void group(int t, int lane) const
    {
        if (t >= O * G) return;
        const int o = t / G, j = t - o * G;
        const float zq = sz[t][1];
        float gs = 0.0f, gz = 0.0f;
        for (int i = j * g + lane; i < (j + 1) * g; i += 32) {
            const size_t e = (size_t)o * I + i;
            const uint32_t *seg = codes + (e & ~(size_t)31) / 32 * BITS;
            gs = __builtin_fmaf(dwhat[e], (float)code_at_rt<BITS>(seg, i & 31) - zq, gs);
            gz += dwhat[e];
        }
        for (int k = 16; k >= 1; k >>= 1) { gs += __shfl_xor(gs, k, 32); gz += __shfl_xor(gz, k, 32); }
        if (lane != 0) return;
        if (ds != nullptr) ds[t] = gs;
        if (dz != nullptr) dz[t] = -sz[t][0] * gz;
    }
};
template <typename E> __global__ __launch_bounds__(256) void k_f32_epilogue(E epi)
{
    epi.group(blockIdx.x * 8 + (threadIdx.x >> 5), threadIdx.x & 31);
}

// ---- a backward of few tiles in two launches ---------------------------------------------------------------
// dX needs What, the gradients of the weights need dWhat, and neither needs the other: dWhat tiles and What in the first launch,
// dX tiles and the per-group epilogue in the second.  What bounds such a call is launches, not work: each of the four in a row took
// 3.6 to 6.5 us whatever it did (256 tokens, 512 x 512, 4 bit, g = 128; forward and backward 27.4 us with four launches in the
// backward, 20.9 with two, before the loads ahead in f32_tile).  The tiles come first, they take longer.
template <typename W>
__global__ __launch_bounds__(512) void k_f32_dwhat_and_what(ColMajorF32 dY, ColMajorF32 X, float *__restrict__ dwhat, int O, int I, int T, uint32_t tiles_n,
                                                            uint32_t tiles, W w, float *__restrict__ what)
{
    __shared__ F32Sums<8, true> sums;
    if (blockIdx.x < tiles) {
        f32_tile<ColMajorF32, ColMajorF32, 1, 1, 8, true>(dY, X, dwhat, O, I, T, false, blockIdx.x % tiles_n, blockIdx.x / tiles_n, sums);
        return;
    }
    f32_what(w, what, (int64_t)(blockIdx.x - tiles) * 512 + threadIdx.x);
}
template <typename E>
__global__ __launch_bounds__(512) void k_f32_dx_and_epilogue(RowMajorF32 dY, ColMajorF32 what, float *__restrict__ dX, int T, int I, int O, uint32_t tiles_n,
                                                             uint32_t tiles, E epi)
{
    __shared__ F32Sums<8, true> sums;
    if (blockIdx.x < tiles) {
        f32_tile<RowMajorF32, ColMajorF32, 1, 1, 8, true>(dY, what, dX, T, I, O, false, blockIdx.x % tiles_n, blockIdx.x / tiles_n, sums);
        return;
    }
    epi.group((blockIdx.x - tiles) * 16 + (threadIdx.x >> 5), threadIdx.x & 31);
}

// ---- host ------------------------------------------------------------------------------------------
template <typename OpA, typename OpB>
static void gemm(OpA a, OpB b, float *C, int M, int N, int K, hipStream_t st)
{
    if (M <= 0 || N <= 0) return;
    // 64 x 64 per wave reads half as much per product; 32 x 32 until that still gives every compute unit a workgroup.  A contraction
    // shorter than the waves' share leaves waves idle that only wait for the sums: with one block of 32 every wave takes a
    // tile of its own (2048 x 2048, 4 bit, g = 32, one token: dWhat and its sums 49 -> 29 us), with two a workgroup has two
    // waves (33 tokens: 48 -> 38; with 256 tiles to go around four are 6 % faster, with three blocks 20 %).
    const int64_t big = ((M + 63) / 64) * (int64_t)((N + 63) / 64);
    const int blocks = (K + 31) / 32;
    const bool along_m = M >= N;
    auto go = [&](auto kernel, int side, int waves, bool split) {
        const int wm = !split && along_m ? waves : 1, wn = !split && !along_m ? waves : 1;
        const dim3 grid((N + side * wn - 1) / (side * wn), (M + side * wm - 1) / (side * wm));
        kernel<<<grid, dim3(64 * waves), 0, st>>>(a, b, C, M, N, K, along_m);
    };
    if (big < 256) go(k_f32_gemm<OpA, OpB, 1, 1, 8, true>, 32, 8, true);
    else if (blocks <= 1) go(k_f32_gemm<OpA, OpB, 2, 2, 4, false>, 64, 4, false);
    else if (blocks == 2 && big >= 512) go(k_f32_gemm<OpA, OpB, 2, 2, 2, true>, 64, 2, true);
    else go(k_f32_gemm<OpA, OpB, 2, 2, 4, true>, 64, 4, true);
}
static RowMajorF32 rows_of(const void *p, int rows, int cols) { return RowMajorF32{(const float *)p, rows, cols, (uint32_t)((size_t)rows * cols * 4)}; }
static ColMajorF32 cols_of(const void *p, int rows, int cols) { return ColMajorF32{(const float *)p, rows, cols}; }

// `what`: scratch for O * I floats
template <typename AccW>
static void dx(const Problem &p, const void *dY, AccW w, float *dX, float *what, hipStream_t st)
{
    const int T = (int)p.T, I = (int)p.I, O = (int)p.O;
    if (O <= kShortO) {
        const int64_t tiles = (int64_t)((T + 63) / 64) * ((I + 63) / 64);
        k_f32_dx_short<AccW><<<dim3((unsigned)tiles), dim3(256), 0, st>>>((const float *)dY, w, dX, T);
        return;
    }
    k_f32_what<AccW><<<dim3((unsigned)(((int64_t)O * (I / 16) + 255) / 256)), dim3(256), 0, st>>>(w, what);
    gemm(rows_of(dY, T, O), ColMajorF32{what, O, I}, dX, T, I, O, st);
}

// f(weights, epilogue) with the types of this call
template <typename F>
static void with_types(const Problem &p, bool block_ap, const void *Wc, const float *s, const void *zsz, const float *dwhat, void *dW, float *ds, float *dz, F &&f)
{
    const int O = (int)p.O, I = (int)p.I, g = (int)p.g, G = (int)p.G;
    if (block_ap) {
        const float qmax = (float)((1 << p.bits) - 1), *const z = (const float *)zsz;
        if (p.w_bf16) f(FakeQuantW<bf16_t>{(const bf16_t *)Wc, s, z, O, I, g, G, qmax}, EpilogueBlockAp<bf16_t>{dwhat, (const bf16_t *)Wc, s, z, (bf16_t *)dW, ds, dz, O, I, g, G, qmax});
        else f(FakeQuantW<float>{(const float *)Wc, s, z, O, I, g, G, qmax}, EpilogueBlockAp<float>{dwhat, (const float *)Wc, s, z, (float *)dW, ds, dz, O, I, g, G, qmax});
    } else {
        const uint32_t *c = (const uint32_t *)Wc; const floatx2 *sz = (const floatx2 *)zsz;
        if (p.bits == 2) f(PackedW<2>{c, sz, O, I, g, G}, EpilogueE2e<2>{dwhat, c, sz, ds, dz, O, I, g, G});
        else if (p.bits == 3) f(PackedW<3>{c, sz, O, I, g, G}, EpilogueE2e<3>{dwhat, c, sz, ds, dz, O, I, g, G});
        else f(PackedW<4>{c, sz, O, I, g, G}, EpilogueE2e<4>{dwhat, c, sz, ds, dz, O, I, g, G});
    }
}

void launch_f32_fwd(const Problem &p, bool packed, const void *X, const void *Wc, const float *s, const void *zsz, void *Y, hipStream_t st)
{
    const int T = (int)p.T, I = (int)p.I, O = (int)p.O;
    with_types(p, !packed, Wc, s, zsz, nullptr, nullptr, nullptr, nullptr, [&](auto w, auto) {
        gemm(rows_of(X, T, I), WeightRows<decltype(w)>{w}, (float *)Y, T, O, I, st);
    });
}

// Both GEMMs of the backward on 32 x 32 tiles (see gemm()), and a dX that reads What from memory.
static bool two_launches(const Problem &p)
{
    const int64_t to = (p.O + 63) / 64, ti = (p.I + 63) / 64, tt = (p.T + 63) / 64;
    return p.T > 0 && p.O > kShortO && tt * ti < 256 && to * ti < 256;
}
size_t f32_what_bytes(const Problem &p) { return two_launches(p) ? (size_t)p.O * p.I * 4 : 0; }

void launch_f32_bwd(const Problem &p, bool block_ap, const void *X, const void *dY, const void *Wc, const float *s, const void *zsz,
                    float *dwhat, float *what, void *dX, void *dW, float *ds, float *dz, hipStream_t st)
{
    const int O = (int)p.O, I = (int)p.I, T = (int)p.T;
    const bool want_w = dW != nullptr || ds != nullptr || dz != nullptr;
    with_types(p, block_ap, Wc, s, zsz, dwhat, dW, ds, dz, [&](auto w, auto epi) {
        typedef decltype(w) W;
        typedef decltype(epi) E;
        const unsigned groups = (unsigned)((size_t)O * p.G);
        if (want_w && dX != nullptr && what != nullptr && two_launches(p)) {
            const unsigned tn = (unsigned)((I + 31) / 32), dw_tiles = tn * (unsigned)((O + 31) / 32), dx_tiles = tn * (unsigned)((T + 31) / 32);
            const unsigned what_blocks = (unsigned)(((int64_t)O * (I / 16) + 511) / 512);
            k_f32_dwhat_and_what<W><<<dim3(dw_tiles + what_blocks), dim3(512), 0, st>>>(cols_of(dY, T, O), cols_of(X, T, I), dwhat, O, I, T, tn, dw_tiles, w, what);
            k_f32_dx_and_epilogue<E><<<dim3(dx_tiles + (groups + 15) / 16), dim3(512), 0, st>>>(rows_of(dY, T, O), ColMajorF32{what, O, I}, (float *)dX, T, I, O, tn, dx_tiles, epi);
            return;
        }
        if (dX != nullptr && T > 0) dx(p, dY, w, (float *)dX, dwhat, st);
        if (!want_w) return;
        // dWhat[o][i] = sum_t dY[t][o] * X[t][i]
        gemm(cols_of(dY, T, O), cols_of(X, T, I), dwhat, O, I, T, st);
        k_f32_epilogue<E><<<dim3((groups + 7) / 8), dim3(256), 0, st>>>(epi);
    });
}

}  // namespace eqat
