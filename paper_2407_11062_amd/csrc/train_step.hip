// Block-AP step glue (Sec. 3.2: a block is trained against its full-precision counterpart with a reconstruction loss;
// Sec. 4.1 "Training": one learning rate for the quantization parameters, another for the weights).  The paper names
// neither the loss form nor the optimizer; mean squared error and AdamW are taken.  Both kernels are streaming passes
// bound by HBM, all arithmetic in binary32.  Of large tensors, what they read is read once and what the update writes is next read a step later, hundreds
// of MB on: non-temporal accesses (one block of 4096 / 11008, fp32 W, 5.7 GB: update 1094 -> 970 us, 5.2 -> 5.8 TB/s; a plain copy by such loads and
// stores reaches 6.2, by others 5.7).  dY, which the backward reads next, is stored as any other tensor (the loss of 8192 x 4096, 201 MB: 51 -> 34 us).
#include "common.h"
#include "kernels.h"

namespace eqat {
namespace {

constexpr int kThreads = 256;
constexpr int kLossBlocksMax = 2048;    // partial sums of the loss; also the length of the workspace in floats

// ONCE: past the caches
template <bool ONCE, typename V> __device__ __forceinline__ V load_v(const V *p)
{
    if constexpr (ONCE) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool ONCE, typename V> __device__ __forceinline__ void store_v(V v, V *p)
{
    if constexpr (ONCE) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <bool ONCE> __device__ __forceinline__ void load8(const float *p, float (&v)[8])
{
    const floatx4 a = load_v<ONCE>(reinterpret_cast<const floatx4 *>(p)), b = load_v<ONCE>(reinterpret_cast<const floatx4 *>(p) + 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) { v[k] = a[k]; v[4 + k] = b[k]; }
}
template <bool ONCE> __device__ __forceinline__ void load8(const bf16_t *p, float (&v)[8])
{
    const uintx4 u = load_v<ONCE>(reinterpret_cast<const uintx4 *>(p));
#pragma unroll
    for (int k = 0; k < 4; ++k) { v[2 * k] = __uint_as_float(u[k] << 16); v[2 * k + 1] = __uint_as_float(u[k] & 0xFFFF0000u); }
}
__device__ __forceinline__ void store8(float *p, const float (&v)[8])
{
    floatx4 a, b;
#pragma unroll
    for (int k = 0; k < 4; ++k) { a[k] = v[k]; b[k] = v[4 + k]; }
    reinterpret_cast<floatx4 *>(p)[0] = a;
    reinterpret_cast<floatx4 *>(p)[1] = b;
}
__device__ __forceinline__ void store8(bf16_t *p, const float (&v)[8])
{
    bf16x8 o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = (bf16_t)v[k];          // round to nearest even
    *reinterpret_cast<bf16x8 *>(p) = o;
}
template <bool ONCE> __device__ __forceinline__ void load4(const float *p, float (&v)[4])
{
    const floatx4 a = load_v<ONCE>(reinterpret_cast<const floatx4 *>(p));
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = a[k];
}
template <bool ONCE> __device__ __forceinline__ void load4(const bf16_t *p, float (&v)[4])
{
    const uintx2 u = load_v<ONCE>(reinterpret_cast<const uintx2 *>(p));
#pragma unroll
    for (int k = 0; k < 2; ++k) { v[2 * k] = __uint_as_float(u[k] << 16); v[2 * k + 1] = __uint_as_float(u[k] & 0xFFFF0000u); }
}
template <bool ONCE> __device__ __forceinline__ void store4(float *p, const float (&v)[4])
{
    const floatx4 a = {v[0], v[1], v[2], v[3]};
    store_v<ONCE>(a, reinterpret_cast<floatx4 *>(p));
}
template <bool ONCE> __device__ __forceinline__ void store4(bf16_t *p, const float (&v)[4])
{
    bf16x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = (bf16_t)v[k];          // round to nearest even
    store_v<ONCE>(__builtin_bit_cast(uintx2, o), reinterpret_cast<uintx2 *>(p));
}
__device__ __forceinline__ void store1(float *p, float v) { *p = v; }
__device__ __forceinline__ void store1(bf16_t *p, float v) { *p = (bf16_t)v; }

// Sum over the workgroup in a fixed order (lanes by xor butterfly, then the waves in order); valid in thread 0.
__device__ __forceinline__ float block_sum(float v)
{
    __shared__ float wave_sum[kThreads / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) t += wave_sum[w];
    }
    return t;
}

// partial[b] = sum over the elements of workgroup b of (Y - Yref)^2;  dY = (Y - Yref) * two_over_n  (dY may be NULL)
template <typename T, bool ONCE>
__global__ __launch_bounds__(kThreads) void k_recon_loss(const T *__restrict__ Y, const T *__restrict__ R, T *__restrict__ dY,
                                                         float *__restrict__ partial, int64_t n, float two_over_n)
{
    const int64_t n8 = n >> 3;
    float acc = 0.f;
    for (int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x; c < n8; c += (int64_t)gridDim.x * kThreads) {
        float y[8], r[8];
        load8<ONCE>(Y + 8 * c, y);
        load8<ONCE>(R + 8 * c, r);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            y[k] -= r[k];
            acc = fmaf(y[k], y[k], acc);
            y[k] *= two_over_n;
        }
        if (dY != nullptr) store8(dY + 8 * c, y);
    }
    // the last n % 8 elements: one each for the first lanes of workgroup 0
    if (blockIdx.x == 0 && (int64_t)threadIdx.x < (n & 7)) {
        const int64_t e = 8 * n8 + threadIdx.x;
        const float d = to_float(Y[e]) - to_float(R[e]);
        acc = fmaf(d, d, acc);
        if (dY != nullptr) store1(dY + e, d * two_over_n);
    }
    const float t = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// loss = (sum of the partials, in a fixed order) / n
__global__ __launch_bounds__(kThreads) void k_recon_finish(const float *__restrict__ partial, int n_partial, float *__restrict__ loss,
                                                           float inv_n)
{
    float acc = 0.f;
    for (int k = threadIdx.x; k < n_partial; k += kThreads) acc += partial[k];
    const float t = block_sum(acc);
    if (threadIdx.x == 0) loss[0] = t * inv_n;
}

// ---- AdamW ---------------------------------------------------------------------------------------------------------
struct AdamSeg {
    void *p; const void *g; float *m; float *v;
    int64_t n;
    float lr, decay;                    // decay = lr * weight_decay
    float p_min;                        // the updated parameter is held at or above this (-inf: no bound)
    uint32_t first_block;
    int32_t bf16;                       // dtype of p and g
};
struct AdamArgs {
    AdamSeg seg[3];                     // W, s, z (n = 0: absent)
    float b1, b2, omb1, omb2, eps, c1, c2;   // omb = 1 - b;  c1 = 1 / (1 - b1^step), c2 = 1 / (1 - b2^step)
};

__device__ __forceinline__ void adam_one(float &p, float g, float &m, float &v, const AdamSeg &sg, const AdamArgs &a)
{
    p -= sg.decay * p;
    m = a.b1 * m + a.omb1 * g;
    v = a.b2 * v + a.omb2 * g * g;
    p -= sg.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
    p = fmaxf(p, sg.p_min);
}

// Workgroup `block` of a parameter tensor: 4 elements per lane and access, neighbouring lanes neighbouring 16 bytes of each fp32 array.
// The last workgroup keeps to that: element by element, eight trips of it, small tensors took up to 1.1 us more (4352 -> 120, 2 bit, 6.2 -> 4.8 us; 1152 -> 104, 4 bit, 4.3 -> 3.4).
constexpr int kAdamUnroll = 2;
template <typename T, bool ONCE>
__device__ __forceinline__ void adam_block(const AdamSeg &sg, const AdamArgs &a, int64_t first)
{
    T *P = static_cast<T *>(sg.p);
    const T *G = static_cast<const T *>(sg.g);
    if (first + 4 * kThreads * kAdamUnroll <= sg.n) {
        float p[kAdamUnroll][4], g[kAdamUnroll][4], m[kAdamUnroll][4], v[kAdamUnroll][4];
#pragma unroll
        for (int u = 0; u < kAdamUnroll; ++u) {
            const int64_t e0 = first + 4 * (u * kThreads + (int)threadIdx.x);
            load4<ONCE>(P + e0, p[u]); load4<ONCE>(G + e0, g[u]); load4<ONCE>(sg.m + e0, m[u]); load4<ONCE>(sg.v + e0, v[u]);
        }
#pragma unroll
        for (int u = 0; u < kAdamUnroll; ++u) {
            const int64_t e0 = first + 4 * (u * kThreads + (int)threadIdx.x);
#pragma unroll
            for (int k = 0; k < 4; ++k) adam_one(p[u][k], g[u][k], m[u][k], v[u][k], sg, a);
            store4<ONCE>(P + e0, p[u]); store4<ONCE>(sg.m + e0, m[u]); store4<ONCE>(sg.v + e0, v[u]);
        }
    } else {
        // the last workgroup of a tensor: whole accesses, then what is left of four elements
#pragma unroll
        for (int u = 0; u < kAdamUnroll; ++u) {
            const int64_t e0 = first + 4 * (u * kThreads + (int)threadIdx.x);
            if (e0 + 4 <= sg.n) {
                float p[4], g[4], m[4], v[4];
                load4<ONCE>(P + e0, p); load4<ONCE>(G + e0, g); load4<ONCE>(sg.m + e0, m); load4<ONCE>(sg.v + e0, v);
#pragma unroll
                for (int k = 0; k < 4; ++k) adam_one(p[k], g[k], m[k], v[k], sg, a);
                store4<ONCE>(P + e0, p); store4<ONCE>(sg.m + e0, m); store4<ONCE>(sg.v + e0, v);
            } else {
                for (int64_t e = e0; e < sg.n; ++e) {
                    float p = to_float(P[e]), m = sg.m[e], v = sg.v[e];
                    adam_one(p, to_float(G[e]), m, v, sg, a);
                    store1(P + e, p); sg.m[e] = m; sg.v[e] = v;
                }
            }
        }
    }
}

// One launch updates the weights, the step sizes and the zero points of a linear: workgroups
// [seg[i].first_block, seg[i+1].first_block) own parameter group i.
template <bool ONCE>
__global__ __launch_bounds__(kThreads) void k_adamw(AdamArgs a)
{
    const int si = blockIdx.x >= a.seg[2].first_block ? 2 : blockIdx.x >= a.seg[1].first_block ? 1 : 0;
    const AdamSeg sg = si == 2 ? a.seg[2] : si == 1 ? a.seg[1] : a.seg[0];     // selects, not a dynamic index
    const int64_t first = (int64_t)(blockIdx.x - sg.first_block) * (4 * kThreads * kAdamUnroll);
    if (sg.bf16) adam_block<bf16_t, ONCE>(sg, a, first);
    else adam_block<float, ONCE>(sg, a, first);
}

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + 4 * kThreads * kAdamUnroll - 1) / (4 * kThreads * kAdamUnroll)); }

// From where on the accesses go past the caches.  Below, an array is still there when its next reader comes.  Graph replays over three states, us, with the
// caches / past them: AdamW, 75 MB (p, g, m, v) 28.1 / 31.0, 100 MB 40.5 / 38.3 (fp32 37.6 / 37.1), 134 MB 55.4 / 47.4; loss, Y and Yref 34 MB 16.7 / 18.1, 67 MB
// 26.2 / 25.6, 134 MB 47.2 / 42.0.  (fp32 activations, whose lanes read 16 of every 32 bytes per instruction, do not gain: 67 MB 47.0 / 47.1.)
constexpr int64_t kAdamOnceBytes = (int64_t)88 << 20, kLossOnceBytes = (int64_t)48 << 20;

}  // namespace

size_t recon_loss_ws_bytes() { return (size_t)kLossBlocksMax * sizeof(float); }

void launch_recon_loss(int64_t n, bool bf16, const void *Y, const void *Yref, float *loss, void *dY, float *partial,
                       hipStream_t st)
{
    const int64_t want = (n / 8 + kThreads - 1) / kThreads;
    const int nb = (int)(want < 1 ? 1 : want > kLossBlocksMax ? kLossBlocksMax : want);
    const float two_over_n = (float)(2.0 / (double)n), inv_n = (float)(1.0 / (double)n);
#define EQAT_LOSS(T, ONCE) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_recon_loss<T, ONCE>), dim3(nb), dim3(kThreads), 0, st, static_cast<const T *>(Y), \
                                              static_cast<const T *>(Yref), static_cast<T *>(dY), partial, n, two_over_n)
    if (!bf16) EQAT_LOSS(float, false);
    else if (n * 4 > kLossOnceBytes) EQAT_LOSS(bf16_t, true);
    else EQAT_LOSS(bf16_t, false);
#undef EQAT_LOSS
    hipLaunchKernelGGL(k_recon_finish, dim3(1), dim3(kThreads), 0, st, partial, nb, loss, inv_n);
}

void launch_adamw(const AdamGroup *groups, float beta1, float beta2, float eps, int step, hipStream_t st)
{
    AdamArgs a{};
    uint32_t first = 0;
    int64_t bytes = 0;
    for (int i = 0; i < 3; ++i) {
        const AdamGroup &gr = groups[i];
        AdamSeg &sg = a.seg[i];
        sg.p = gr.p; sg.g = gr.g; sg.m = gr.m; sg.v = gr.v;
        sg.n = gr.p != nullptr ? gr.n : 0;
        sg.lr = gr.lr; sg.decay = (float)((double)gr.lr * (double)gr.weight_decay);
        sg.first_block = first; sg.bf16 = gr.bf16 ? 1 : 0; sg.p_min = gr.p_min;
        first += blocks_for(sg.n);
        bytes += sg.n * (gr.bf16 ? 12 : 16);
    }
    if (first == 0) return;
    a.b1 = beta1; a.b2 = beta2; a.omb1 = (float)(1.0 - (double)beta1); a.omb2 = (float)(1.0 - (double)beta2); a.eps = eps;
    a.c1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    a.c2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    if (bytes > kAdamOnceBytes) hipLaunchKernelGGL(k_adamw<true>, dim3(first), dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL(k_adamw<false>, dim3(first), dim3(kThreads), 0, st, a);
}

}  // namespace eqat
