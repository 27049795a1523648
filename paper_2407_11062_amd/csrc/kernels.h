// Internal launcher interface between the C ABI (api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/eqat.h"

namespace eqat {

struct Problem {
    int64_t T, I, O, g, G;
    int bits;
    bool act_bf16, w_bf16;
};

// ---- quant.hip -------------------------------------------------------------------------------
// Eq.(1): W,s,z -> codes (+ optional clamp bit-plane [O,I/8] bytes, + optional (s,zbar) pairs [O,G]).
// for_pack: the dense stream of the C ABI; otherwise the working layout the GEMM kernels read (work_code_bytes()).
// zpacked (may be NULL): the zero points at N bits are packed by extra workgroups of the same launch.
// zero_words (may be NULL): n_zero 32-bit words that the launch also clears (the arrival counters of the GEMMs).
void launch_quantize(const Problem &p, const void *W, const float *s, const float *z, void *codes, void *clampbits,
                     void *sz, void *zpacked, bool for_pack, uint32_t *zero_words, uint32_t n_zero, hipStream_t st);
// The same for up to kMaxBatch matrices in ONE launch; all jobs share bits, the weight dtype, and whether a clamp plane
// is written (the first job decides).
constexpr int kMaxBatch = EQAT_MAX_BATCH;
struct QuantizeJob {
    Problem p; const void *W; const float *s, *z; void *codes, *clampbits, *sz, *zpacked; uint32_t *zero_words; uint32_t n_zero;
};
void launch_quantize_batch(const QuantizeJob *jobs, int n, bool for_pack, hipStream_t st);
struct InitJob { Problem p; const void *W; float *s, *z; };
void launch_init_minmax_batch(const InitJob *jobs, int n, hipStream_t st);       // all jobs share bits and the weight dtype
inline size_t work_code_bytes(const Problem &p) { return (size_t)p.O * p.I / (p.bits == 2 ? 4 : 2); }
// One launch before the GEMMs of an E2E-QP call: dense stream -> working layout (packed == NULL: skipped) and the
// (s, z) pairs (sz == NULL: skipped), z taken from the packed N-bit zero points or from a float array (exactly one of
// the two not NULL); zb_out (may be NULL) receives the zero points alone, as floats.
void launch_e2e_prepare(const Problem &p, const void *packed, void *work, const float *s, const void *zpacked,
                        const float *zfloat, void *sz, float *zb_out, uint32_t *zero_words, uint32_t n_zero, hipStream_t st);
// Test aid: working-layout codes -> int32 [O,I]; clamp bit-plane -> bytes 0/1 [O,I]; (s, zero point) pairs -> the
// zero points [O,G] (each output may be NULL).
void launch_unpack_work(const Problem &p, const void *work, const void *clampbits, const void *sz, int32_t *codes,
                        uint8_t *clamped, float *zbar, hipStream_t st);
void launch_unpack(const Problem &p, const void *Wpacked, const void *zpacked, int32_t *codes, int32_t *zcodes, hipStream_t st);
void launch_init_minmax(const Problem &p, const void *W, float *s, float *z, hipStream_t st);
// ds / dz (each may be NULL) of n_out groups from n_per consecutive partials each; dz is scaled by -s.
void launch_reduce_partials(const float *part_ds, const float *part_dz, float *ds, float *dz, const float *s, size_t n_out,
                            uint32_t n_per, hipStream_t st);

// ---- gemm_mfma.hip (bf16 activations) -----------------------------------------------------------
// Scratch of the GEMM launches that cut the tiles of a partly filled last round along K: one buffer of fp32 accumulator
// tiles and one arrival counter per tile.  The counters must be zero when a launch starts; every launch leaves them zero.
// Either pointer NULL, or too few bytes for what a plan would write: tiles are not cut.
struct SkScratch { float *partials; size_t bytes; uint32_t *counters; };
int plan_item_for_test(const Problem &p, int gemm, int block, int j, int32_t item[12]);      // test aid, see gemm_mfma.hip
// Test aid: bytes from sk.partials on within which the launch of a GEMM (0 fwd, 1 dX, 2 dW) on a device of `cus` compute units writes.
size_t parts_written_for_test(const Problem &p, int gemm, int cus, const SkScratch &sk);
void dx_route_for_test(const Problem &p, bool block_ap, int32_t route[2]);      // test aid, see eqat_dx_route
// Bytes of that scratch for the launches of a forward that takes the tile kernels (fwd), a backward (bwd), or both.  *partial_bytes: what their plans write;
// *needed_bytes: what a call cannot do without: launches that share tiles only to fill the chip run unshared in less.
void sk_scratch_bytes(const Problem &p, bool fwd, bool bwd, size_t *partial_bytes, size_t *needed_bytes, size_t *counter_bytes);
// Y[T,O] = X[T,I] * What[O,I]^T with What = (code - zbar) * s rebuilt per tile from packed codes.
void launch_mfma_fwd(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, const SkScratch &sk,
                     hipStream_t st);
// dX[T,I] = dY[T,O] * What[O,I]
void launch_mfma_dx(const Problem &p, const void *dY, const void *codes, const void *sz, void *dX, const SkScratch &sk,
                    hipStream_t st);
// dWhat = dY^T X fused with the per-element / per-group epilogue.
//   block_ap: needs W, clampbits; writes dW (W's dtype, may be NULL), ds, dz (may be NULL).
//   e2e_qp  : W = clampbits = dW = NULL; writes ds and, if not NULL, dz = -s * group-sum dWhat.
// `part` is scratch for [2][O, I/32] floats, used only when a group is wider than one tile (see dw_needs_partials);
// `sk` is the scratch of launches that cut tiles along T.
void launch_mfma_dw(const Problem &p, bool block_ap, const void *X, const void *dY, const void *W, const void *codes,
                    const void *clampbits, const void *sz, const float *s, void *dW, float *ds, float *dz, float *part,
                    const SkScratch &sk, hipStream_t st);
bool dw_needs_partials(const Problem &p);
// Both of them (dX, or all of dW, ds and dz, may be NULL: the other alone), in one launch where that is faster.
void launch_mfma_bwd(const Problem &p, bool block_ap, const void *X, const void *dY, const void *W, const void *codes,
                     const void *clampbits, const void *sz, const float *s, void *dX, void *dW, float *ds, float *dz, float *part,
                     const SkScratch &sk, hipStream_t st);

// The kernel that a forward with bf16 activations takes, and the piece of the output that a workgroup of it computes (0: the
// tile kernel plans that by itself).
enum FwdKernel { FWD_TILES, FWD_MID, FWD_GEMV_WIDE, FWD_GEMV_ANY, FWD_GEMV_RUN, FWD_GEMV_RUN_SEGMENTS, FWD_GEMV_RUN_PAIRS,
                 FWD_RELAY_MID /* the codes re-laid, then FWD_MID from the working layout */ };
struct FwdRoute { FwdKernel kernel; int tokens, rows; };

// ---- gemv.hip (E2E-QP forward for a few tokens, straight from the dense packed stream) -----------
bool gemv_applies(const Problem &p);
FwdRoute gemv_route(const Problem &p, bool floatz);         // where one of the two predicates holds
// The same on the working layout and the (s, z) pairs, bitwise the same results: calls that hold those take it where this applies.
bool gemv_work_applies(const Problem &p);
void launch_gemv_work(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, hipStream_t st);
// exactly one of zpacked / zfloat is not NULL
void launch_gemv(const Problem &p, const void *X, const void *Wpacked, const float *s, const void *zpacked,
                 const float *zfloat, void *Y, hipStream_t st);

// whether mulhi(segment, ceil(2^32 / (g / 32))) is the group of every segment of a row
inline bool group_by_magic(const Problem &p) { return (p.I / 32) * (p.g / 32) < ((int64_t)1 << 32); }

// ---- gemm_ksplit.hip (fwd / dX on codes in the working layout, few 128 x 128 output tiles) --------------------
// Workgroups that share a tile of the forward (bt = false) or dX (bt = true); 0: the tile kernels of gemm_mfma.hip compute it.
int ksplit_parts(const Problem &p, bool bt, const SkScratch &sk);
size_t ksplit_bytes(const Problem &p, bool bt, int parts);          // of sk.partials; 0 for one part
bool ksplit_item_for_test(const Problem &p, bool bt, const SkScratch &sk, int block, int32_t item[10]);      // test aid
void launch_ksplit(const Problem &p, bool bt, const void *A, const void *codes, const void *sz, void *C, const SkScratch &sk,
                   int parts, hipStream_t st);

// ---- gemm_mid.hip (forward for few output tiles) --------------------------------------------
bool mid_applies(const Problem &p);
FwdRoute mid_route(const Problem &p, bool from_packed);
double mid_us(const Problem &p);                  // what it takes, as the rules of dispatch estimate it
// from the caller's dense stream (exactly one of zpacked / zfloat is not NULL), or from the working layout and (s, z) pairs:
// bitwise the same results
void launch_mid(const Problem &p, const void *X, const void *Wpacked, const float *s, const void *zpacked, const float *zfloat,
                void *Y, hipStream_t st);
void launch_mid_work(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, hipStream_t st);
// the same from the working layout, step sizes and zero points (O * G floats each); leaves them as pairs for a backward (`pairs` NULL: does not)
bool mid_pairs_itself(const Problem &p, bool keep);       // where that is faster than a small launch that makes the pairs in front
void launch_mid_prepared(const Problem &p, const void *X, const void *codes, const float *s, const float *z, void *pairs, void *Y, hipStream_t st);

// ---- gemm_mid_dx.hip (dX for few output tiles, on codes in the working layout) -------------------------
double mid_dx_us(const Problem &p, int cus, int *tokens);      // what it takes, as the rule of dispatch estimates it, and with which token tiles; 1e30: too many tiles
void launch_mid_dx(const Problem &p, int tokens, const void *dY, const void *codes, const void *sz, void *dX, hipStream_t st);

// ---- train_step.hip (Block-AP step glue: reconstruction loss, AdamW over {W, s, z}) --------------------
size_t recon_loss_ws_bytes();
// loss[0] = mean (Y - Yref)^2, dY (may be NULL) = 2 (Y - Yref) / n; `partial` = recon_loss_ws_bytes() of scratch.
void launch_recon_loss(int64_t n, bool bf16, const void *Y, const void *Yref, float *loss, void *dY, float *partial,
                       hipStream_t st);
struct AdamGroup {                      // one parameter tensor; p == NULL: absent
    void *p; const void *g; float *m; float *v;
    int64_t n;
    float lr, weight_decay;
    bool bf16;                          // dtype of p and g (moments are always fp32)
    float p_min;                        // lower bound of the updated parameter (-inf: none)
};
// One launch over three parameter groups (weights, step sizes, zero points); step counts from 1.
void launch_adamw(const AdamGroup *groups, float beta1, float beta2, float eps, int step, hipStream_t st);

// ---- gemm_f32.hip (fp32 activations; binary32 products and sums, exact division everywhere) --------
void launch_f32_fwd(const Problem &p, bool packed, const void *X, const void *W_or_codes, const float *s, const void *z_or_sz,
                    void *Y, hipStream_t st);
// What a backward asks for beside the O*I floats of `dwhat` to run in two launches instead of four (0: it does not).
size_t f32_what_bytes(const Problem &p);
// dX (may be NULL) = dY What; dWhat[O,I] = dY^T X into `dwhat` (scratch of O*I floats), then the per-group epilogue into dW, ds, dz (each may be
// NULL).  `what`: f32_what_bytes() of scratch, or NULL.
void launch_f32_bwd(const Problem &p, bool block_ap, const void *X, const void *dY, const void *W_or_codes, const float *s,
                    const void *z_or_sz, float *dwhat, float *what, void *dX, void *dW, float *ds, float *dz, hipStream_t st);

}  // namespace eqat
