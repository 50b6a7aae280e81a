// Internal declarations shared by the translation units of libnm_mvue (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define NM_DT_F32 0
#define NM_DT_BF16 1
#define NM_DT_F32_BF16X3 2   // update GEMM only: binary32 operands, multiplied as three bf16 terms each

namespace nm {

// Output scale of the 8-bit update GEMM: a host value, or (inv_a != nullptr) value * inv_a[1] * inv_b[1] with the two
// factors read on the device -- element [1] of a scale record written by launch_q8_scale is the inverse scale.  The kernels
// multiply them; for the 384 x 256 one the launcher leaves the product in inv_b[3] (the record's scratch slot).
struct AlphaArg {
    float value;
    const float *inv_a, *inv_b;
    AlphaArg(float v = 1.0f, const float *a = nullptr, const float *b = nullptr) : value(v), inv_a(a), inv_b(b) {}
};

hipError_t launch_prune(int dt, int m, int est, const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed,
                        uint32_t stream_id, void *vals, uint16_t *meta, void *dense, int64_t ldd, hipStream_t st);

// prune fused into the producer of the neural gradient: g_l = u * d (eq. (2): d = f'(z_l), u = W^T g_{l+1}) is written
// dense to gout and pruned + compressed in the same pass
hipError_t launch_prune_producer(int dt, int m, int est, const void *u, int64_t ldu, const void *d, int64_t ldd, int64_t T, int64_t O,
                                 uint64_t seed, uint32_t stream_id, void *gout, int64_t ldgo, void *vals, uint16_t *meta, hipStream_t st);

// the same prunes for a gradient stored transposed: gT [O x T], row stride ldt (est 0 optimal 2:4, 1 approx-MVUE 2:4, 3 MVUE 1:2)
hipError_t launch_prune_transposed(int dt, int est, const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed,
                                   uint32_t stream_id, void *vals, uint16_t *meta, hipStream_t st);

// approx-MVUE 4:8 (four magnitude-proportional draws out of eight): vals [T/2 x O] in octet order, meta32 [T/16 x O]
hipError_t launch_prune_4of8_approx(int dt, const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed, uint32_t stream_id,
                                    void *vals, uint32_t *meta32, void *dense, int64_t ldd, hipStream_t st);

hipError_t launch_compress(int dt, int m, const void *d, int64_t T, int64_t O, int64_t ld, void *vals,
                           uint16_t *meta, int32_t *bad, hipStream_t st);

// dW = beta*dW + decompress(vals, meta)^T h
hipError_t launch_update_gemm(int dt, const void *vals, const uint16_t *meta, const void *h, int64_t ldh,
                              float *dW, int64_t lddw, int64_t T, int64_t O, int64_t I, float beta,
                              void *workspace, size_t workspace_bytes, hipStream_t st);
size_t update_gemm_workspace(int dt, int64_t T, int64_t O, int64_t I);

// kernels behind launch_update_gemm: sparse MFMA for bf16, dense fp32 MFMA for binary32; both split the reduction
// axis into slabs for shapes with few output tiles and sum the partials with launch_splitk_reduce
hipError_t launch_update_gemm_smfmac(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, float *dW,
                                     int64_t lddw, int64_t T, int64_t O, int64_t I, float beta, void *workspace,
                                     hipStream_t st);
size_t update_gemm_smfmac_workspace(int64_t T, int64_t O, int64_t I, size_t beside = 0);     // beside: workspace bytes of the call that are not partial sums
// small problems (gemm_smfmac_small.hip): slabs partial sums of groups_per_slab (even) token groups each, slab_stride apart; h_rows rows of h (at most T, the rest count as zeros)
hipError_t launch_update_gemm_smfmac_small(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, int64_t h_rows, float *out, int64_t ldo,
                                           int64_t slab_stride, int slabs, int64_t groups_per_slab, int64_t T, int64_t O, int64_t I, int accumulate, hipStream_t st);
// the same for 8-bit operands; groups of 32 tokens; alpha scales what is stored
hipError_t launch_update_gemm_q8_small(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *h8, int64_t ldh, float *out, int64_t ldo, int64_t slab_stride,
                                       int slabs, int64_t groups_per_slab, int64_t T, int64_t O, int64_t I, int accumulate, const AlphaArg &alpha, hipStream_t st);
size_t update_gemm_smfmac_shifted_workspace(int64_t T, int64_t O, int64_t I);
// the same product with h given as n row-shifted views of one [rows x cb] matrix x (bf16): h[t][j*cb + c] = x[(t + rows[j])*ldx + c]
hipError_t launch_update_gemm_smfmac_shifted(const void *vals, const uint16_t *meta, const void *x, int64_t ldx, int64_t cb,
                                             const int64_t *rows, int n, float *dW, int64_t lddw, int64_t T, int64_t O,
                                             float beta, void *workspace, hipStream_t st);
hipError_t launch_update_gemm_f32(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, float *dW,
                                  int64_t lddw, int64_t T, int64_t O, int64_t I, float beta, void *workspace,
                                  hipStream_t st);
size_t update_gemm_f32_workspace(int64_t T, int64_t O, int64_t I);

// binary32 operands split into three bf16 terms each, six partial products on the sparse 16-bit path (gemm_f32_split.hip)
hipError_t launch_update_gemm_f32_split(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, float *dW,
                                        int64_t lddw, int64_t T, int64_t O, int64_t I, float beta, void *workspace,
                                        hipStream_t st);
size_t update_gemm_f32_split_workspace(int64_t T, int64_t O, int64_t I);
// A second pass over the slabs of n4 float4 sums: from 12 slabs on a sum runs as eight chains, which eight threads take (`shared`) or one thread
// side by side; either way in the same order.
enum class SlabSum { one_chain, eight_chains, shared };
SlabSum slab_sum_form(int64_t n4, int slabs);
hipError_t launch_splitk_reduce(const float *part, int slabs, float *dW, int64_t lddw, int64_t O, int64_t I,
                                int accumulate, AlphaArg alpha, hipStream_t st);

// 8-bit path: 2:4 prune with e5m2 output (stochastic rounding) in 32-token groups, and its update GEMM
// dW = beta*dW + alpha * decompress(vals8, meta32)^T h8  (vals8 e5m2, h8 e4m3)
hipError_t launch_prune_q8(int dt, int est, const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed,
                           uint32_t stream_id, float scale, const float *scale_dev, uint8_t *vals8, uint32_t *meta32, hipStream_t st);
// ... of a gradient stored transposed (gT [O x T], tokens contiguous)
hipError_t launch_prune_q8_transposed(int dt, int est, const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed,
                                      uint32_t stream_id, float scale, const float *scale_dev, uint8_t *vals8, uint32_t *meta32,
                                      hipStream_t st);
hipError_t launch_update_gemm_q8(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *h8, int64_t ldh, float *dW,
                                 int64_t lddw, int64_t T, int64_t O, int64_t I, AlphaArg alpha, float beta, void *workspace,
                                 hipStream_t st);
size_t update_gemm_q8_workspace(int64_t T, int64_t O, int64_t I);
// ... with h8 given as n row-shifted views of one [rows x cb] matrix x8
hipError_t launch_update_gemm_q8_shifted(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *x8, int64_t ldx, int64_t cb,
                                         const int64_t *rows, int n, float *dW, int64_t lddw, int64_t T, int64_t O,
                                         AlphaArg alpha, float beta, void *workspace, hipStream_t st);
size_t update_gemm_q8_shifted_workspace(int64_t T, int64_t O, int64_t I);

// 8-bit path, per-tensor scale and activation cast (q8_scale.hip).  rec: device float[4] = {s, 1/s, bits of max|t|, 0}
// with s the largest power of two such that s * max|t| <= top (1 for an all-zero or non-finite tensor).
hipError_t launch_q8_scale(int dt, const void *t, int64_t R, int64_t C, int64_t ld, float top, float *rec, hipStream_t st);
// A tensor's scale inside a layer's call: the maxima of the n workgroups that passed over it (LAYER_PEAKS words of workspace, aligned to 16
// bytes), the format's top, and the record that the first kernel to use the scale leaves for those behind it
constexpr int LAYER_PEAKS = 256;
struct LayerScale { uint32_t *peaks; int n; float top; float *rec; };
// the maxima of a layer's two bf16 tensors (R x C, row stride ld; not empty) in one launch, into s0 and s1, whose n it sets
hipError_t launch_layer_peaks(const void *t0, int64_t R0, int64_t C0, int64_t ld0, LayerScale &s0, const void *t1, int64_t R1, int64_t C1, int64_t ld1,
                              LayerScale &s1, hipStream_t st);
// h8 = e4m3(h * rec[0]), round to nearest even, magnitudes beyond 448 saturate
hipError_t launch_cast_e4m3(int dt, const void *h, int64_t R, int64_t C, int64_t ld, const float *rec, uint8_t *h8, int64_t ld8,
                            hipStream_t st);
// measurement aid: streams 64 KB in and 36 KB out per block (the 16-bit prune's read:write mix)
hipError_t launch_rw_mix_probe(const void *src, void *dst, int64_t n_blocks, hipStream_t st);

// ---- layers (nm_layers.hip): a k x k, stride-1, "same" convolution on bf16 tensors [N, C, H, W] / [N, O, H, W], each stored
// as channel planes or channels last
struct ConvShape { int N, C, O, H, W, k; bool x_channels_last, g_channels_last; };
// one launch: rows [-margin, out_rows - margin) of the zero-padded channels-last grid of the activations, as bf16 (sx == nullptr) or
// e4m3(x * its scale), and the 2:4 prune (est 0 optimal, 1 approx-MVUE) of the gradient on that grid, T rows; sg: 8-bit
// output in 32-token groups
hipError_t launch_grid(const ConvShape &cs, const void *x, int64_t margin, int64_t out_rows, const LayerScale *sx, void *x_out, int est,
                       const void *gy, int64_t T, uint64_t seed, uint32_t stream_id, const LayerScale *sg, void *vals, void *meta, hipStream_t st);

// The update GEMMs without their second pass: binary32 partial sums part[slabs][O][I], at most parts_bytes of them (one
// slab where the plan has no split); the caller sums them with launch_finish.
size_t update_gemm_smfmac_shifted_parts_bytes(int64_t T, int64_t O, int64_t I);
hipError_t launch_update_gemm_smfmac_shifted_parts(const void *vals, const uint16_t *meta, const void *x, int64_t ldx, int64_t cb,
                                                   const int64_t *rows, int n, int64_t T, int64_t O, float *part, int *slabs, hipStream_t st);
size_t update_gemm_q8_shifted_parts_bytes(int64_t T, int64_t O, int64_t I);
hipError_t launch_update_gemm_q8_shifted_parts(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *x8, int64_t ldx, int64_t cb,
                                               const int64_t *rows, int n, int64_t T, int64_t O, float *part, int *slabs, hipStream_t st);
// 3 x 3 convolutions with all taps of a channel block in one workgroup (gemm_conv.hip)
struct ConvGemmPlan {
    int64_t T, x_rows;                    // tokens (the grid's rows rounded up) and rows of the activations' buffer, whatever its last ones hold
    int slabs;                            // partial sums: [slabs][O][9][C]
};
bool conv_gemm_plan(const ConvShape &cs, bool q8, ConvGemmPlan &p);       // false: not a case of it
hipError_t launch_conv_gemm(const ConvShape &cs, bool q8, const ConvGemmPlan &p, const void *vals, const void *meta, const void *x_full,
                            float *part, hipStream_t st);
// conv weight gradient, bf16 [O][C][taps] = alpha * sum over the slabs of part[slabs][O][taps][C]
hipError_t launch_finish_conv(const float *part, int slabs, void *dW, int64_t O, int C, int taps, AlphaArg alpha, hipStream_t st);

// ... of a linear layer (bf16 tensors, T tokens, not necessarily whole token groups)
constexpr int64_t LAYER_LD_MOST = (int64_t)1 << 21;       // largest row stride, in elements: the prune's offsets inside a wave are 32 bits wide
hipError_t launch_prune_layer(int m, int est, const void *g, int64_t ldg, const void *act, int64_t lda, int64_t T, int64_t O, uint64_t seed,
                              uint32_t stream_id, void *gout, int64_t ldgo, void *vals, uint16_t *meta, float *csum, hipStream_t st);
hipError_t launch_prune_q8_layer(int est, const void *g, int64_t ldg, int64_t T, int64_t O, uint64_t seed, uint32_t stream_id,
                                 const LayerScale &ls, uint8_t *vals8, uint32_t *meta32, float *csum, hipStream_t st);
hipError_t launch_cast_e4m3_layer(const void *h, int64_t R, int64_t C, int64_t ld, const LayerScale &ls, uint8_t *h8, int64_t ld8, int64_t out_rows,
                                  hipStream_t st);
hipError_t launch_pad_rows(const void *h, int64_t rows, int64_t C, int64_t ld, void *out, int64_t out_rows, hipStream_t st);
size_t update_gemm_smfmac_parts_bytes(int64_t h_rows, int64_t T, int64_t O, int64_t I, bool *needs_whole_rows);
hipError_t launch_update_gemm_smfmac_parts(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, int64_t h_rows, int64_t T,
                                           int64_t O, int64_t I, bool whole_rows, float *part, int *slabs, hipStream_t st);
size_t update_gemm_q8_parts_bytes(int64_t T, int64_t O, int64_t I);
hipError_t launch_update_gemm_q8_parts(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *h8, int64_t ldh, int64_t T, int64_t O,
                                       int64_t I, float *part, int *slabs, hipStream_t st);
// dW (bf16, contiguous [O][I]) = alpha * sum of the slabs; db (bf16 [O], may be null) = sum of the groups' column sums
hipError_t launch_finish_linear(const float *part, int slabs, int64_t O, int64_t I, void *dW, AlphaArg alpha, const float *csum, int64_t groups,
                                void *db, hipStream_t st);

// The dense products of a linear layer (gemm_dense.hip): y[M x N] = x[M x K] w^T + bias, w [N][K] contiguous, bias and ReLU optional; nn: w is
// [K][N] and y = x w.  bf16, N and K multiples of 8
hipError_t launch_dense_gemm(bool nn, const void *x, int64_t ldx, const void *w, const void *bias, void *y, int64_t ldy, int64_t M, int64_t N, int64_t K,
                             bool relu, hipStream_t st);

// The library's static device scratch array (nm_static.hip): its size, and its address on the current device
// (looked up once per device; no allocation).
size_t static_scratch_bytes();
hipError_t static_scratch(void **ptr);

}  // namespace nm
