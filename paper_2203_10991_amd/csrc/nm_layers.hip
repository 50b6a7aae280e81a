// C ABI of the layer entry points: argument checks, the layout of their workspace, the sequence of launches.
// Every check runs before any device work; no allocation, no synchronisation.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/nm_mvue.h"
#include "nm_internal.h"

namespace nm { int abi_fail(int code, const char *message); void abi_clear(); }      // nm_last_error()'s slot (nm_abi.hip)

namespace {

int fail(int code, const char *fmt, ...)
{
    char text[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(text, sizeof text, fmt, ap);
    va_end(ap);
    return nm::abi_fail(code, text);
}
int launched(const char *fn, hipError_t e)
{
    if (e != hipSuccess) return fail(NM_ERR_LAUNCH, "%s: HIP launch failed: %s", fn, hipGetErrorString(e));
    nm::abi_clear();
    return NM_OK;
}
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }
inline bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return na && nb && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}
// parts of a workspace, one after the other on 256-byte boundaries
struct Carver {
    size_t used = 0;
    size_t take(size_t bytes) { const size_t at = used; used += (bytes + 255) / 256 * 256; return at; }
};

// the two scales of a call with 8-bit operands: maxima, then the records
constexpr size_t SCALES = 2 * nm::LAYER_PEAKS * 4 + 32;
nm::LayerScale scale_at(char *scales, int which, float top)
{
    return nm::LayerScale{(uint32_t *)scales + which * nm::LAYER_PEAKS, 0, top, (float *)(scales + 2 * nm::LAYER_PEAKS * 4) + which * 4};
}

struct ConvPlan {
    nm::ConvShape cs;
    int64_t T, margin, I;
    bool taps;                            // the nine-tap kernel; otherwise the general update GEMM on shifted views
    nm::ConvGemmPlan gemm;
    size_t x_full, vals, meta, recs, part, bytes;
};
ConvPlan plan_conv(const nm::ConvShape &cs, bool q8)
{
    ConvPlan p;
    p.cs = cs;
    const int pad = cs.k / 2;
    const int64_t Wp = cs.W + 2 * pad, rows = (int64_t)cs.N * (cs.H + 2 * pad) * Wp, gt = q8 ? 32 : 16;
    p.taps = nm::conv_gemm_plan(cs, q8, p.gemm);
    p.T = p.taps ? p.gemm.T : (rows + gt - 1) / gt * gt;
    p.margin = pad * Wp + pad;
    p.I = (int64_t)cs.C * cs.k * cs.k;
    Carver c;
    p.recs = c.take(q8 ? SCALES : 0);
    p.x_full = c.take((size_t)(p.taps ? p.gemm.x_rows : p.T + 2 * p.margin) * cs.C * (q8 ? 1 : 2));
    p.vals = c.take((size_t)(p.T / 2) * cs.O * (q8 ? 1 : 2));
    p.meta = c.take((size_t)(p.T / gt) * cs.O * (q8 ? 4 : 2));
    p.part = c.take(p.taps ? (size_t)p.gemm.slabs * cs.O * p.I * sizeof(float)
                    : q8 ? nm::update_gemm_q8_shifted_parts_bytes(p.T, cs.O, p.I) : nm::update_gemm_smfmac_shifted_parts_bytes(p.T, cs.O, p.I));
    p.bytes = c.used;
    return p;
}
// sizes a convolution call accepts (checked before anything is computed from them)
const char *bad_conv_shape(int64_t N, int64_t C, int64_t O, int64_t H, int64_t W, int k, int q8)
{
    const int64_t lim = (int64_t)1 << 20;
    if (N < 1 || C < 1 || O < 1 || H < 1 || W < 1 || N > lim || C > lim || O > lim || H > lim || W > lim) return "every size must be in 1..2^20";
    if (k != 1 && k != 3 && k != 5) return "the kernel must be 1, 3 or 5 wide";
    if (O % 8 || C % (q8 ? 16 : 8)) return "O must be a multiple of 8 and C of 8 (16 with 8-bit operands)";
    const int64_t Hp = H + k, Wp = W + k, cmax = C > O ? C : O, rows_lim = ((int64_t)1 << 31) - 65536;
    if (N > rows_lim / Hp / Wp || (Wp * k + 1024) * C > (1ll << 30)) return "the padded grid exceeds what 32-bit row numbers and byte offsets reach";
    if (N * Hp * Wp > ((int64_t)1 << 58) / cmax) return "a tensor is larger than 2^58 elements";
    return nullptr;
}

struct LinearPlan {
    int64_t Tp, groups;                   // tokens rounded up to whole groups of 16 (8-bit: 32)
    bool copy_h;                          // h is copied with zero rows up to Tp
    size_t recs, h, vals, meta, csum, part, bytes;
};
LinearPlan plan_linear(int64_t T, int64_t O, int64_t I, bool q8, bool bias)
{
    LinearPlan p;
    const int64_t gt = q8 ? 32 : 16;
    p.Tp = (T + gt - 1) / gt * gt;
    p.groups = p.Tp / gt;
    bool whole = false;
    const size_t part = q8 ? nm::update_gemm_q8_parts_bytes(p.Tp, O, I) : nm::update_gemm_smfmac_parts_bytes(T, p.Tp, O, I, &whole);
    p.copy_h = !q8 && whole && p.Tp != T;
    Carver c;
    p.recs = c.take(q8 ? SCALES : 0);
    p.h = c.take(q8 ? (size_t)p.Tp * I : p.copy_h ? (size_t)p.Tp * I * 2 : 0);
    p.vals = c.take((size_t)(p.Tp / 2) * O * (q8 ? 1 : 2));
    p.meta = c.take((size_t)p.groups * O * (q8 ? 4 : 2));
    p.csum = c.take(bias ? (size_t)p.groups * O * 4 : 0);
    p.part = c.take(part);
    p.bytes = c.used;
    return p;
}
const char *bad_linear_shape(int64_t T, int64_t O, int64_t I, int q8)
{
    const int64_t lim = (int64_t)1 << 21;
    if (T < 1 || O < 1 || I < 1 || O > lim || I > lim || T > ((int64_t)1 << 34) / O || T > ((int64_t)1 << 36) / I)
        return "sizes must be positive, O and I at most 2^21, T * O at most 2^34 and T * I at most 2^36";
    if (O % 8 || I % (q8 ? 16 : 8)) return "O must be a multiple of 8 and I of 8 (16 with 8-bit operands)";
    return nullptr;
}

}  // namespace

// y = x w^T (+ bias, ReLU) or, nn, y = x w: checks of the two dense products of a linear layer
static int dense_checked(const char *fn, bool nn, const void *x, int64_t ldx, const void *w, const void *bias, void *y, int64_t M, int64_t N, int64_t K,
                         bool relu, void *hip_stream)
{
    const int64_t T = M, O = nn ? K : N, I = nn ? N : K;
    if (const char *why = bad_linear_shape(T, O, I, 0)) return fail(NM_ERR_SHAPE, "%s: %s", fn, why);
    if (!x || !w || !y) return fail(NM_ERR_NULL, "%s: a tensor is NULL", fn);
    if (ldx < K || ldx > nm::LAYER_LD_MOST) return fail(NM_ERR_SHAPE, "%s: a row stride is smaller than its row or beyond 2^21", fn);
    if (!aligned16(x) || !aligned16(w) || !aligned16(bias) || !aligned16(y) || ldx % 8)
        return fail(NM_ERR_ALIGN, "%s: bases and row strides need 16-byte alignment", fn);
    const size_t yb = (size_t)M * N * 2, xb = (size_t)((M - 1) * ldx + K) * 2, wb = (size_t)O * I * 2, bb = bias ? (size_t)N * 2 : 0;
    if (overlap(y, yb, x, xb) || overlap(y, yb, w, wb) || overlap(y, yb, bias, bb)) return fail(NM_ERR_ALIAS, "%s: the output overlaps an input", fn);
    return launched(fn, nm::launch_dense_gemm(nn, x, ldx, w, bias, y, N, M, N, K, relu, (hipStream_t)hip_stream));
}

extern "C" {

int nm_linear_forward(const void *x, int64_t ldx, const void *w, const void *bias, int64_t T, int64_t O, int64_t I, int relu, void *y, void *hip_stream)
{
    return dense_checked("nm_linear_forward", false, x, ldx, w, bias, y, T, O, I, relu != 0, hip_stream);
}

int nm_linear_input_grad(const void *g, int64_t ldg, const void *w, int64_t T, int64_t O, int64_t I, void *dx, void *hip_stream)
{
    return dense_checked("nm_linear_input_grad", true, g, ldg, w, nullptr, dx, T, I, O, false, hip_stream);
}

size_t nm_linear_update_workspace(int64_t T, int64_t O, int64_t I, int q8, int bias)
{
    if (bad_linear_shape(T, O, I, q8)) return 0;
    return plan_linear(T, O, I, q8 != 0, bias != 0).bytes;
}

int nm_linear_update(const void *g, int64_t ldg, const void *act, int64_t lda, const void *h, int64_t ldh, int64_t T, int64_t O, int64_t I,
                     int m, int mode, int q8, uint64_t seed, uint32_t stream_id, void *g_out, int64_t ldgo, void *dW, void *db,
                     void *workspace, size_t workspace_bytes, void *hip_stream)
{
    const char *fn = "nm_linear_update";
    if (m != 2 && m != 4) return fail(NM_ERR_UNSUPPORTED, "%s: blocks of %d (2 = MVUE 1:2, 4 = MVUE 2:4)", fn, m);
    if (mode != 0 && !(mode == 1 && m == 4)) return fail(NM_ERR_UNSUPPORTED, "%s: unknown mode %d (0 = optimal MVUE, 1 = approx-MVUE 2:4)", fn, mode);
    if (act && q8) return fail(NM_ERR_UNSUPPORTED, "%s: the 8-bit form takes the gradient itself, not a ReLU's output beside it", fn);
    if (const char *why = bad_linear_shape(T, O, I, q8)) return fail(NM_ERR_SHAPE, "%s: %s", fn, why);
    if (!g || !h || !dW || (act && !g_out)) return fail(NM_ERR_NULL, "%s: g, h, dW (and g_out with act) must not be NULL", fn);
    const int64_t lim = nm::LAYER_LD_MOST;
    if (ldg < O || ldh < I || ldg > lim || ldh > lim || (act && (lda < O || ldgo < O || lda > lim || ldgo > lim)))
        return fail(NM_ERR_SHAPE, "%s: a row stride is smaller than its row or beyond 2^21", fn);
    if (!aligned16(g) || !aligned16(h) || !aligned16(dW) || !aligned16(db) || !aligned16(workspace) || ldg % 8 || ldh % 8 ||
        (act && (!aligned16(act) || !aligned16(g_out) || lda % 8 || ldgo % 8)))
        return fail(NM_ERR_ALIGN, "%s: bases and row strides need 16-byte alignment", fn);
    const LinearPlan p = plan_linear(T, O, I, q8 != 0, db != nullptr);
    if (!workspace || workspace_bytes < p.bytes)
        return fail(NM_ERR_WORKSPACE, "%s: workspace of %zu bytes required, %zu given", fn, p.bytes, workspace ? workspace_bytes : (size_t)0);
    struct { const void *p; size_t n; } in[3] = {{g, (size_t)((T - 1) * ldg + O) * 2}, {h, (size_t)((T - 1) * ldh + I) * 2},
                                                 {act, act ? (size_t)((T - 1) * lda + O) * 2 : 0}},
                                        out[4] = {{dW, (size_t)O * I * 2}, {db, db ? (size_t)O * 2 : 0},
                                                  {g_out, act ? (size_t)((T - 1) * ldgo + O) * 2 : 0}, {workspace, p.bytes}};
    for (int i = 0; i < 4; ++i) {
        for (int j = 0; j < 3; ++j) if (overlap(out[i].p, out[i].n, in[j].p, in[j].n)) return fail(NM_ERR_ALIAS, "%s: an output overlaps an input", fn);
        for (int j = 0; j < i; ++j) if (overlap(out[i].p, out[i].n, out[j].p, out[j].n)) return fail(NM_ERR_ALIAS, "%s: two outputs overlap", fn);
    }

    hipStream_t st = (hipStream_t)hip_stream;
    char *w = (char *)workspace;
    float *part = (float *)(w + p.part), *csum = db ? (float *)(w + p.csum) : nullptr;
    hipError_t e = hipSuccess;
    int slabs = 1;
    nm::AlphaArg alpha(1.0f);
    if (q8) {
        nm::LayerScale sg = scale_at(w + p.recs, 0, 57344.0f / (float)m), sh = scale_at(w + p.recs, 1, 448.0f);
        e = nm::launch_layer_peaks(g, T, O, ldg, sg, h, T, I, ldh, sh, st);
        if (e == hipSuccess) e = nm::launch_cast_e4m3_layer(h, T, I, ldh, sh, (uint8_t *)(w + p.h), I, p.Tp, st);
        if (e == hipSuccess)
            e = nm::launch_prune_q8_layer(m == 2 ? 3 : mode, g, ldg, T, O, seed, stream_id, sg, (uint8_t *)(w + p.vals), (uint32_t *)(w + p.meta), csum, st);
        if (e == hipSuccess)
            e = nm::launch_update_gemm_q8_parts((const uint8_t *)(w + p.vals), (const uint32_t *)(w + p.meta), (const uint8_t *)(w + p.h), I, p.Tp, O, I,
                                                part, &slabs, st);
        alpha = nm::AlphaArg(1.0f, sg.rec, sh.rec);
    } else {
        if (p.copy_h) e = nm::launch_pad_rows(h, T, I, ldh, w + p.h, p.Tp, st);
        if (e == hipSuccess)
            e = nm::launch_prune_layer(m, mode, g, ldg, act, lda, T, O, seed, stream_id, g_out, ldgo, w + p.vals, (uint16_t *)(w + p.meta), csum, st);
        if (e == hipSuccess)
            e = nm::launch_update_gemm_smfmac_parts(w + p.vals, (const uint16_t *)(w + p.meta), p.copy_h ? w + p.h : h, p.copy_h ? I : ldh,
                                                    p.copy_h ? p.Tp : T, p.Tp, O, I, T == p.Tp, part, &slabs, st);
    }
    if (e == hipSuccess) e = nm::launch_finish_linear(part, slabs, O, I, dW, alpha, csum, p.groups, db, st);
    return launched(fn, e);
}

size_t nm_conv_update_workspace(int64_t N, int64_t C, int64_t O, int64_t H, int64_t W, int k, int q8)
{
    if (bad_conv_shape(N, C, O, H, W, k, q8)) return 0;
    return plan_conv(nm::ConvShape{(int)N, (int)C, (int)O, (int)H, (int)W, k, false, false}, q8 != 0).bytes;
}

int nm_conv_update(const void *gy, int gy_channels_last, const void *x, int x_channels_last, int64_t N, int64_t C, int64_t O, int64_t H,
                   int64_t W, int k, int q8, int mode, uint64_t seed, uint32_t stream_id, void *dW, void *workspace, size_t workspace_bytes,
                   void *hip_stream)
{
    const char *fn = "nm_conv_update";
    if (mode != 0 && mode != 1) return fail(NM_ERR_UNSUPPORTED, "%s: unknown mode %d (0 = optimal MVUE, 1 = approx-MVUE)", fn, mode);
    if (const char *why = bad_conv_shape(N, C, O, H, W, k, q8)) return fail(NM_ERR_SHAPE, "%s: %s", fn, why);
    if (!gy || !x || !dW) return fail(NM_ERR_NULL, "%s: gy, x and dW must not be NULL", fn);
    if (!aligned16(gy) || !aligned16(x) || !aligned16(dW) || !aligned16(workspace))
        return fail(NM_ERR_ALIGN, "%s: gy, x, dW and the workspace need 16-byte aligned bases", fn);
    const nm::ConvShape cs{(int)N, (int)C, (int)O, (int)H, (int)W, k, x_channels_last != 0, gy_channels_last != 0};
    const ConvPlan p = plan_conv(cs, q8 != 0);
    if (!workspace || workspace_bytes < p.bytes)
        return fail(NM_ERR_WORKSPACE, "%s: workspace of %zu bytes required, %zu given", fn, p.bytes, workspace ? workspace_bytes : (size_t)0);
    const int64_t gn = N * O * H * W, xn = N * C * H * W;
    const size_t gb = (size_t)gn * 2, xb = (size_t)xn * 2, wb = (size_t)O * p.I * 2;
    if (overlap(dW, wb, gy, gb) || overlap(dW, wb, x, xb) || overlap(workspace, p.bytes, gy, gb) || overlap(workspace, p.bytes, x, xb) ||
        overlap(workspace, p.bytes, dW, wb))
        return fail(NM_ERR_ALIAS, "%s: dW and the workspace must not overlap an input or each other", fn);

    hipStream_t st = (hipStream_t)hip_stream;
    char *w = (char *)workspace;
    nm::LayerScale sg = scale_at(w + p.recs, 0, 57344.0f / 4.0f), sx = scale_at(w + p.recs, 1, 448.0f);
    float *part = (float *)(w + p.part);
    int64_t shifts[32];
    const int pad = k / 2, Wp = (int)W + 2 * pad;
    for (int ky = 0; ky < k; ++ky)
        for (int kx = 0; kx < k; ++kx) shifts[ky * k + kx] = (int64_t)(ky - pad) * Wp + (kx - pad);
    hipError_t e = hipSuccess;
    int slabs = 1;
    nm::AlphaArg alpha(1.0f);
    if (q8) {
        // (the border's zeros do not change a maximum: the scales are those of the tensors as they are)
        e = nm::launch_layer_peaks(gy, 1, gn, gn, sg, x, 1, xn, xn, sx, st);
        alpha = nm::AlphaArg(1.0f, sg.rec, sx.rec);
    }
    if (e == hipSuccess)
        e = nm::launch_grid(cs, x, p.margin, p.T + 2 * p.margin, q8 ? &sx : nullptr, w + p.x_full, mode, gy, p.T, seed, stream_id,
                            q8 ? &sg : nullptr, w + p.vals, w + p.meta, st);
    const char *x0 = w + p.x_full + p.margin * C * (q8 ? 1 : 2);
    if (e == hipSuccess && p.taps) {
        slabs = p.gemm.slabs;
        e = nm::launch_conv_gemm(cs, q8 != 0, p.gemm, w + p.vals, w + p.meta, w + p.x_full, part, st);
    } else if (e == hipSuccess)
        e = q8 ? nm::launch_update_gemm_q8_shifted_parts((const uint8_t *)(w + p.vals), (const uint32_t *)(w + p.meta), (const uint8_t *)x0, C, C,
                                                         shifts, k * k, p.T, O, part, &slabs, st)
               : nm::launch_update_gemm_smfmac_shifted_parts(w + p.vals, (const uint16_t *)(w + p.meta), x0, C, C, shifts, k * k, p.T, O, part,
                                                             &slabs, st);
    if (e == hipSuccess) e = nm::launch_finish_conv(part, slabs, dW, O, (int)C, k * k, alpha, st);
    return launched(fn, e);
}

}  // extern "C"
