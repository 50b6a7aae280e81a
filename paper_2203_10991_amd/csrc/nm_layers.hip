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

struct ConvPlan {
    nm::ConvShape cs;
    int64_t T, margin, I;
    size_t x_full, vals, meta, recs, part, bytes;
};
ConvPlan plan_conv(const nm::ConvShape &cs, bool q8)
{
    ConvPlan p;
    p.cs = cs;
    const int pad = cs.k / 2;
    const int64_t Wp = cs.W + 2 * pad, rows = (int64_t)cs.N * (cs.H + 2 * pad) * Wp, gt = q8 ? 32 : 16;
    p.T = (rows + gt - 1) / gt * gt;
    p.margin = pad * Wp + pad;
    p.I = (int64_t)cs.C * cs.k * cs.k;
    Carver c;
    p.recs = c.take(32);
    p.x_full = c.take((size_t)(p.T + 2 * p.margin) * cs.C * (q8 ? 1 : 2));
    p.vals = c.take((size_t)(p.T / 2) * cs.O * (q8 ? 1 : 2));
    p.meta = c.take((size_t)(p.T / gt) * cs.O * (q8 ? 4 : 2));
    p.part = c.take(q8 ? nm::update_gemm_q8_shifted_parts_bytes(p.T, cs.O, p.I) : nm::update_gemm_smfmac_shifted_parts_bytes(p.T, cs.O, p.I));
    p.bytes = c.used;
    return p;
}
// sizes a convolution call accepts (checked before anything is computed from them)
const char *bad_conv_shape(int64_t N, int64_t C, int64_t O, int64_t H, int64_t W, int k, int q8)
{
    const int64_t lim = (int64_t)1 << 20;
    if (N < 1 || C < 1 || O < 1 || H < 1 || W < 1 || N > lim || C > lim || O > lim || H > lim || W > lim) return "every size must be in 1..2^20";
    if (k < 1 || k % 2 == 0 || k * k > 32) return "the kernel must be odd, with at most 32 taps";
    if (O % 8 || C % (q8 ? 16 : 8)) return "O must be a multiple of 8 and C of 8 (16 with 8-bit operands)";
    const int64_t Hp = H + k, Wp = W + k, cmax = C > O ? C : O, rows_lim = ((int64_t)1 << 31) - 65536;
    if (N > rows_lim / Hp / Wp || (Wp * k + 1024) * C > (1ll << 30)) return "the padded grid exceeds what 32-bit row numbers and byte offsets reach";
    if (N * Hp * Wp > ((int64_t)1 << 58) / cmax) return "a tensor is larger than 2^58 elements";
    return nullptr;
}

}  // namespace

extern "C" {

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
    float *rec_g = (float *)(w + p.recs), *rec_x = rec_g + 4, *part = (float *)(w + p.part);
    int64_t shifts[32];
    const int pad = k / 2, Wp = (int)W + 2 * pad;
    for (int ky = 0; ky < k; ++ky)
        for (int kx = 0; kx < k; ++kx) shifts[ky * k + kx] = (int64_t)(ky - pad) * Wp + (kx - pad);
    hipError_t e = hipSuccess;
    int slabs = 1;
    nm::AlphaArg alpha(1.0f);
    if (q8) {
        // (the border's zeros do not change a maximum: the scales are those of the tensors as they are)
        e = nm::launch_q8_scale_pair(gy, 1, gn, gn, 57344.0f / 4.0f, rec_g, x, 1, xn, xn, 448.0f, rec_x, st);
        alpha = nm::AlphaArg(1.0f, rec_g, rec_x);
    }
    if (e == hipSuccess) e = nm::launch_grid_pack(cs, x, p.margin, p.T + 2 * p.margin, q8 ? rec_x : nullptr, w + p.x_full, st);
    if (e == hipSuccess) e = nm::launch_prune_grid(cs, mode, gy, p.T, seed, stream_id, q8 ? rec_g : nullptr, w + p.vals, w + p.meta, st);
    const char *x0 = w + p.x_full + p.margin * C * (q8 ? 1 : 2);
    if (e == hipSuccess)
        e = q8 ? nm::launch_update_gemm_q8_shifted_parts((const uint8_t *)(w + p.vals), (const uint32_t *)(w + p.meta), (const uint8_t *)x0, C, C,
                                                         shifts, k * k, p.T, O, part, &slabs, st)
               : nm::launch_update_gemm_smfmac_shifted_parts(w + p.vals, (const uint16_t *)(w + p.meta), x0, C, C, shifts, k * k, p.T, O, part,
                                                             &slabs, st);
    if (e == hipSuccess) e = nm::launch_finish_conv(part, slabs, dW, O, (int)C, k * k, alpha, st);
    return launched(fn, e);
}

}  // extern "C"
