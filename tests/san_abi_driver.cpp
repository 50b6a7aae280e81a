// Sanitizer driver for the host side of the C ABI (test infrastructure): csrc/nm_abi.hip and csrc/nm_layers.hip are compiled for
// the host only under -fsanitize=address,undefined and linked with the stub launchers below instead of the kernels, so the
// argument validation -- everything that runs before a launch -- executes on a machine without a GPU.  The driver
// walks the error paths (null, ragged, misaligned, overlapping, absurdly large arguments: the range arithmetic must
// not overflow) and the accepting paths (on which the stubs read what the real launchers read on the host).
// Run by tests/test_sanitizers.py.  Exit status 0 = every call returned what it should and no sanitizer reported.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "nm_mvue.h"

static int g_launches = 0;
namespace nm {
struct AlphaArg { float value; const float *inv_a, *inv_b; };      // layout of the library's own (passed by value)
hipError_t launch_prune(int, int, int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, void *, uint16_t *, void *, int64_t,
                        hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_producer(int, int, int, const void *, int64_t, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, void *,
                                 int64_t, void *, uint16_t *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_transposed(int, int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, void *, uint16_t *,
                                   hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_4of8_approx(int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, void *, uint32_t *, void *, int64_t,
                                    hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_compress(int, int, const void *, int64_t, int64_t, int64_t, void *, uint16_t *, int32_t *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_q8(int, int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, float, const float *, uint8_t *, uint32_t *,
                           hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_q8_transposed(int, int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, float, const float *, uint8_t *,
                                      uint32_t *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_q8_scale(int, const void *, int64_t, int64_t, int64_t, float, float *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_cast_e4m3(int, const void *, int64_t, int64_t, int64_t, const float *, uint8_t *, int64_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_rw_mix_probe(const void *, void *, int64_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_update_gemm(int, const void *, const uint16_t *, const void *, int64_t, float *, int64_t, int64_t, int64_t, int64_t, float,
                              void *, size_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_update_gemm_q8(const uint8_t *, const uint32_t *, const uint8_t *, int64_t, float *, int64_t, int64_t, int64_t, int64_t,
                                 AlphaArg, float, void *, hipStream_t) { ++g_launches; return hipSuccess; }
static int64_t read_rows(const int64_t *rows, int n) { int64_t s = 0; for (int j = 0; j < n; ++j) s += rows[j]; return s; }
hipError_t launch_update_gemm_smfmac_shifted(const void *, const uint16_t *, const void *, int64_t, int64_t, const int64_t *rows, int n, float *,
                                             int64_t, int64_t, int64_t, float, void *, hipStream_t)
{ ++g_launches; return read_rows(rows, n) == INT64_MIN ? hipErrorUnknown : hipSuccess; }
hipError_t launch_update_gemm_q8_shifted(const uint8_t *, const uint32_t *, const uint8_t *, int64_t, int64_t, const int64_t *rows, int n,
                                         float *, int64_t, int64_t, int64_t, AlphaArg, float, void *, hipStream_t)
{ ++g_launches; return read_rows(rows, n) == INT64_MIN ? hipErrorUnknown : hipSuccess; }
// split-K whenever there are few output tiles, as the real plans do (sizes only matter to the checks)
size_t update_gemm_workspace(int, int64_t T, int64_t O, int64_t I) { return O * I <= 1 << 20 && T >= 1024 ? (size_t)(2 * O * I * 4) : 0; }
size_t update_gemm_q8_workspace(int64_t T, int64_t O, int64_t I) { return update_gemm_workspace(1, T, O, I); }
size_t update_gemm_smfmac_shifted_workspace(int64_t T, int64_t O, int64_t I) { return update_gemm_workspace(1, T, O, I); }
size_t update_gemm_q8_shifted_workspace(int64_t T, int64_t O, int64_t I) { return update_gemm_workspace(1, T, O, I); }
// the layer entry points (nm_layers.hip); the nine-tap plan as the real one's for images it takes
struct ConvShape { int N, C, O, H, W, k; bool x_channels_last, g_channels_last; };
struct ConvGemmPlan { int64_t T, x_rows; int slabs; };
struct LayerScale { uint32_t *peaks; int n; float top; float *rec; };
hipError_t launch_layer_peaks(const void *, int64_t, int64_t, int64_t, LayerScale &, const void *, int64_t, int64_t, int64_t, LayerScale &,
                              hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_cast_e4m3_layer(const void *, int64_t, int64_t, int64_t, const LayerScale &, uint8_t *, int64_t, int64_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_pad_rows(const void *, int64_t, int64_t, int64_t, void *, int64_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_layer(int, int, const void *, int64_t, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, void *, int64_t, void *, uint16_t *,
                              float *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_prune_q8_layer(int, const void *, int64_t, int64_t, int64_t, uint64_t, uint32_t, const LayerScale &, uint8_t *, uint32_t *, float *,
                                 hipStream_t) { ++g_launches; return hipSuccess; }
size_t update_gemm_smfmac_parts_bytes(int64_t h_rows, int64_t T, int64_t O, int64_t I, bool *whole) { *whole = h_rows != T && O >= 1024; return (size_t)(2 * O * I * 4); }
hipError_t launch_update_gemm_smfmac_parts(const void *, const uint16_t *, const void *, int64_t, int64_t, int64_t, int64_t, int64_t, bool, float *, int *slabs,
                                           hipStream_t) { *slabs = 2; ++g_launches; return hipSuccess; }
size_t update_gemm_q8_parts_bytes(int64_t, int64_t O, int64_t I) { return (size_t)(2 * O * I * 4); }
hipError_t launch_update_gemm_q8_parts(const uint8_t *, const uint32_t *, const uint8_t *, int64_t, int64_t, int64_t, int64_t, float *, int *slabs,
                                       hipStream_t) { *slabs = 2; ++g_launches; return hipSuccess; }
hipError_t launch_dense_gemm(bool, const void *, int64_t, const void *, const void *, void *, int64_t, int64_t, int64_t, int64_t, bool, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_finish_linear(const float *, int, int64_t, int64_t, void *, AlphaArg, const float *, int64_t, void *, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_grid(const ConvShape &, const void *, int64_t, int64_t, const LayerScale *, void *, int, const void *, int64_t, uint64_t, uint32_t, const LayerScale *, void *,
                       void *, hipStream_t) { ++g_launches; return hipSuccess; }
bool conv_gemm_plan(const ConvShape &cs, bool, ConvGemmPlan &p)
{
    if (cs.k != 3 || cs.C % 32 || cs.O < 48 || cs.W > 90) return false;
    p.T = ((int64_t)cs.N * (cs.H + 2) * (cs.W + 2) + 127) / 128 * 128; p.x_rows = p.T + 512; p.slabs = 2;
    return true;
}
hipError_t launch_conv_gemm(const ConvShape &, bool, const ConvGemmPlan &, const void *, const void *, const void *, float *, hipStream_t) { ++g_launches; return hipSuccess; }
size_t update_gemm_smfmac_shifted_parts_bytes(int64_t, int64_t O, int64_t I) { return (size_t)(2 * O * I * 4); }
size_t update_gemm_q8_shifted_parts_bytes(int64_t, int64_t O, int64_t I) { return (size_t)(2 * O * I * 4); }
hipError_t launch_update_gemm_smfmac_shifted_parts(const void *, const uint16_t *, const void *, int64_t, int64_t, const int64_t *rows, int n, int64_t, int64_t, float *,
                                                   int *slabs, hipStream_t)
{ *slabs = 2; ++g_launches; return read_rows(rows, n) == INT64_MIN ? hipErrorUnknown : hipSuccess; }
hipError_t launch_update_gemm_q8_shifted_parts(const uint8_t *, const uint32_t *, const uint8_t *, int64_t, int64_t, const int64_t *rows, int n, int64_t, int64_t, float *,
                                               int *slabs, hipStream_t)
{ *slabs = 2; ++g_launches; return read_rows(rows, n) == INT64_MIN ? hipErrorUnknown : hipSuccess; }
hipError_t launch_finish_conv(const float *, int, void *, int64_t, int, int, AlphaArg, hipStream_t) { ++g_launches; return hipSuccess; }
size_t static_scratch_bytes() { return (size_t)32 << 20; }
static char fake_scratch[64];
hipError_t static_scratch(void **p) { *p = fake_scratch; return hipSuccess; }
}  // namespace nm

static int failures = 0;
#define EXPECT(call, code)                                                                                  \
    do {                                                                                                    \
        const int before_ = g_launches;                                                                     \
        const int rc_ = (call);                                                                             \
        if (rc_ != (code)) { fprintf(stderr, "line %d: %s -> %d (%s), wanted %d\n", __LINE__, #call, rc_, nm_last_error(), (int)(code)); ++failures; } \
        if ((code) != 0 && g_launches != before_) { fprintf(stderr, "line %d: launched despite error\n", __LINE__); ++failures; } \
        if ((code) != 0 && !nm_last_error()[0]) { fprintf(stderr, "line %d: no message\n", __LINE__); ++failures; }   \
    } while (0)

int main()
{
    // "device" buffers: host memory of exactly the size the shapes need (never dereferenced by the ABI), 16-byte aligned
    const int64_t T = 1024, O = 64, I = 128;
    std::vector<uint8_t> gbuf(T * O * 4 + 64), vbuf(T / 2 * O * 4 + 64), mbuf(T / 16 * O * 4 + 64), hbuf(T * I * 4 + 64),
        dbuf(T * O * 4 + 64), wbuf(O * I * 4 + 64), wsbuf(2 * O * 144 * 4 + 64), xbuf((T + 64) * I * 2 + 64);
    auto al = [](std::vector<uint8_t> &v) { return (void *)(((uintptr_t)v.data() + 15) & ~(uintptr_t)15); };
    void *g = al(gbuf), *vals = al(vbuf), *meta = al(mbuf), *h = al(hbuf), *dense = al(dbuf), *ws = al(wsbuf), *x = al(xbuf);
    float *dW = (float *)al(wbuf);
    uint16_t *m16 = (uint16_t *)meta;
    uint32_t *m32 = (uint32_t *)meta;
    const size_t wsb = 2 * O * I * 4, wsb_conv = 2 * O * 144 * 4;
    const int64_t huge = (int64_t)1 << 61;

    // ---- accepting paths
    for (int dt = 0; dt < 2; ++dt) {
        EXPECT(mvue_prune_1of2(g, T, O, O, dt, 1, 2, vals, m16, dense, O, nullptr), NM_OK);
        EXPECT(mvue_prune_2of4(g, T, O, O, dt, 1, 2, 0, vals, m16, nullptr, 0, nullptr), NM_OK);
        EXPECT(mvue_prune_2of4(g, T, O, O, dt, 1, 2, 1, vals, m16, dense, O, nullptr), NM_OK);
        EXPECT(mvue_prune_1of4(g, T, O, O, dt, 1, 2, vals, m16, dense, O, nullptr), NM_OK);
        EXPECT(mvue_prune_4of8_approx(g, T, O, O, dt, 1, 2, vals, m32, dense, O, nullptr), NM_OK);
        EXPECT(nm_prune_greedy(g, T, O, O, dt, 2, 4, vals, m16, dense, O, nullptr), NM_OK);
        EXPECT(nm_prune_greedy(g, T, O, O, dt, 1, 2, vals, m16, nullptr, 0, nullptr), NM_OK);
        EXPECT(mvue_prune_2of4_t(g, T, O, T, dt, 1, 2, 0, vals, m16, nullptr), NM_OK);
        EXPECT(mvue_prune_1of2_t(g, T, O, T, dt, 1, 2, vals, m16, nullptr), NM_OK);
        EXPECT(nm_compress(dense, T, O, O, dt, 2, 4, vals, m16, nullptr, nullptr), NM_OK);
        EXPECT(mvue_prune_2of4_q8(g, T, O, O, dt, 1, 2, 0, 0.5f, (uint8_t *)vals, m32, nullptr), NM_OK);
        EXPECT(mvue_prune_1of2_q8(g, T, O, O, dt, 1, 2, 0.5f, (uint8_t *)vals, m32, nullptr), NM_OK);
        EXPECT(mvue_prune_2of4_q8_t(g, T, O, T, dt, 1, 2, 1, 0.5f, nullptr, (uint8_t *)vals, m32, nullptr), NM_OK);
        EXPECT(mvue_prune_1of2_q8_t(g, T, O, T, dt, 1, 2, 0.5f, nullptr, (uint8_t *)vals, m32, nullptr), NM_OK);
        EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, dt, 0.f, ws, wsb, nullptr), NM_OK);
        EXPECT(nm_update_gemm_static(vals, m16, h, I, dW, I, T, O, I, dt, 1.f, nullptr), NM_OK);
    }
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, NM_F32_BF16X3, 0.f, ws, wsb, nullptr), NM_OK);
    EXPECT(nm_update_gemm_q8((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, T, O, I, 1.f, 0.f, ws, wsb, nullptr), NM_OK);
    const int64_t shifts[9] = {-7, -6, -5, -1, 0, 1, 5, 6, 7};
    const int64_t cb = 16;
    void *x0 = (char *)x + 16 * cb * 2;             // row 0 with 16 margin rows before it
    EXPECT(nm_update_gemm_shifted(vals, m16, x0, cb, cb, shifts, 9, dW, 9 * cb, T, O, NM_BF16, 0.f, ws, wsb_conv, nullptr), NM_OK);
    EXPECT(nm_update_gemm_q8_shifted((const uint8_t *)vals, m32, (const uint8_t *)x0, cb, cb, shifts, 9, dW, 9 * cb, T, O, 1.f, 0.f, ws, wsb_conv,
                                     nullptr), NM_OK);
    // prune fused into the producer of g
    EXPECT(mvue_prune_2of4_producer(g, O, h, O, T, O, NM_BF16, 1, 2, 0, dense, O, vals, m16, nullptr), NM_OK);
    EXPECT(mvue_prune_1of2_producer(g, O, h, O, T, O, NM_F32, 1, 2, dense, O, vals, m16, nullptr), NM_OK);
    EXPECT(mvue_prune_2of4_producer(g, O, h, O, T, O, NM_BF16, 1, 2, 3, dense, O, vals, m16, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(mvue_prune_2of4_producer(g, O, nullptr, O, T, O, NM_BF16, 1, 2, 0, dense, O, vals, m16, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_2of4_producer(g, O, h, O, T, O, NM_BF16, 1, 2, 0, g, O, vals, m16, nullptr), NM_ERR_ALIAS);
    EXPECT(mvue_prune_2of4_producer(g, O, h, O, T, O, NM_BF16, 1, 2, 0, dense, O, (char *)h + 64, m16, nullptr), NM_ERR_ALIAS);
    EXPECT(mvue_prune_2of4_producer(g, O, h, O - 8, T, O, NM_BF16, 1, 2, 0, dense, O, vals, m16, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_producer(g, huge, h, huge, huge, O, NM_BF16, 1, 2, 0, dense, huge, vals, m16, nullptr), NM_ERR_SHAPE);
    // device-side scales of the 8-bit path
    alignas(16) static float rec_g[4], rec_h[4];
    EXPECT(nm_q8_scale(g, T, O, O, NM_BF16, 448.f, rec_g, nullptr), NM_OK);
    EXPECT(nm_q8_scale(g, T, O, O, NM_F32, 57344.f / 4.f, rec_h, nullptr), NM_OK);
    EXPECT(nm_cast_e4m3(h, T, I, I, NM_BF16, rec_h, (uint8_t *)x, I, nullptr), NM_OK);
    EXPECT(mvue_prune_2of4_q8_ds(g, T, O, O, NM_BF16, 1, 2, 0, rec_g, (uint8_t *)vals, m32, nullptr), NM_OK);
    EXPECT(mvue_prune_1of2_q8_ds(g, T, O, O, NM_BF16, 1, 2, rec_g, (uint8_t *)vals, m32, nullptr), NM_OK);
    EXPECT(mvue_prune_2of4_q8_t(g, T, O, T, NM_BF16, 1, 2, 0, -1.f, rec_g, (uint8_t *)vals, m32, nullptr), NM_OK);     // the record wins
    EXPECT(mvue_prune_1of2_q8_t(g, T, O, T, NM_BF16, 1, 2, 0.f, rec_g, (uint8_t *)vals, m32, nullptr), NM_OK);
    EXPECT(nm_update_gemm_q8_ds((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, T, O, I, rec_g, rec_h, 0.f, ws, wsb, nullptr), NM_OK);
    EXPECT(nm_update_gemm_q8_shifted_ds((const uint8_t *)vals, m32, (const uint8_t *)x0, cb, cb, shifts, 9, dW, 9 * cb, T, O, rec_g, rec_h, 0.f,
                                        ws, wsb_conv, nullptr), NM_OK);
    EXPECT(nm_q8_scale(g, T, O, O, NM_BF16, 0.f, rec_g, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_q8_scale(g, T, O + 4, O + 4, NM_BF16, 1.f, rec_g, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_q8_scale(g, T, O, O, NM_BF16, 1.f, nullptr, nullptr), NM_ERR_NULL);
    EXPECT(nm_q8_scale(g, T, O, O, NM_BF16, 1.f, (float *)((char *)g + 64), nullptr), NM_ERR_ALIAS);
    EXPECT(nm_q8_scale(g, huge, huge, huge, NM_BF16, 1.f, rec_g, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_cast_e4m3(h, T, I + 8, I + 8, NM_BF16, rec_h, (uint8_t *)x, I + 8, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_cast_e4m3(h, T, I, I, NM_BF16, rec_h, (uint8_t *)h + 32, I, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_cast_e4m3(h, T, I, I, NM_BF16, nullptr, (uint8_t *)x, I, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_2of4_q8_ds(g, T, O, O, NM_BF16, 1, 2, 0, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_2of4_q8_ds(g, T, O, O, NM_BF16, 1, 2, 0, rec_g + 1, (uint8_t *)vals, m32, nullptr), NM_ERR_ALIGN);
    EXPECT(nm_update_gemm_q8_ds((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, T, O, I, rec_g, nullptr, 0.f, ws, wsb, nullptr), NM_ERR_NULL);
    EXPECT(nm_update_gemm_q8_ds((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, T, O, I, dW + 4, rec_h, 0.f, ws, wsb, nullptr), NM_ERR_ALIAS);
    // the read/write-mix probe (pointers are never dereferenced on the host)
    EXPECT(nm_rw_mix_probe(g, (char *)g + (1ll << 40), 3, nullptr), NM_OK);
    EXPECT(nm_rw_mix_probe(g, (char *)g + 65536, 1, nullptr), NM_OK);
    EXPECT(nm_rw_mix_probe(g, (char *)g + 65536, 2, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_rw_mix_probe(g, nullptr, 1, nullptr), NM_ERR_NULL);
    EXPECT(nm_rw_mix_probe((char *)g + 4, (char *)g + (1ll << 40), 1, nullptr), NM_ERR_ALIGN);
    EXPECT(nm_rw_mix_probe(g, g, -1, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_rw_mix_probe(nullptr, nullptr, 0, nullptr), NM_OK);
    // empty problems do nothing and need no pointers
    EXPECT(mvue_prune_2of4(nullptr, 0, O, O, NM_BF16, 0, 0, 0, nullptr, nullptr, nullptr, 0, nullptr), NM_OK);
    EXPECT(mvue_prune_4of8_approx(nullptr, T, 0, 0, NM_BF16, 0, 0, nullptr, nullptr, nullptr, 0, nullptr), NM_OK);
    EXPECT(nm_update_gemm(nullptr, nullptr, nullptr, 0, dW, I, 0, O, I, NM_BF16, 0.f, nullptr, 0, nullptr), NM_OK);
    if (nm_update_gemm_workspace(T, O, I, NM_BF16) != wsb || nm_update_gemm_workspace(-1, O, I, NM_BF16) != 0) ++failures;

    // ---- rejecting paths: one of each kind per family of entry points
    EXPECT(mvue_prune_1of2(nullptr, T, O, O, NM_BF16, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_2of4(g, T, O, O, NM_BF16, 0, 0, 0, nullptr, m16, nullptr, 0, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_2of4(g, T + 4, O, O, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, T, O + 4, O + 4, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, T, O, O - 8, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, -16, O, O, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, T, O, O, 7, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_DTYPE);
    EXPECT(mvue_prune_2of4(g, T, O, O, NM_BF16, 0, 0, 5, vals, m16, nullptr, 0, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(mvue_prune_2of4((char *)g + 2, T, O, O, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_ALIGN);
    EXPECT(mvue_prune_2of4(g, T, O, O + 4, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_ALIGN);
    EXPECT(mvue_prune_2of4(g, T, O, O, NM_BF16, 0, 0, 0, (char *)g + 64, m16, nullptr, 0, nullptr), NM_ERR_ALIAS);
    EXPECT(mvue_prune_2of4(g, T, O, O, NM_BF16, 0, 0, 0, vals, m16, (char *)vals + 16, O, nullptr), NM_ERR_ALIAS);
    EXPECT(mvue_prune_4of8_approx(g, T, O, O, NM_BF16, 0, 0, vals, (uint32_t *)((char *)vals + 32), nullptr, 0, nullptr), NM_ERR_ALIAS);
    EXPECT(mvue_prune_4of8_approx(g, T + 8, O, O, NM_BF16, 0, 0, vals, m32, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_prune_greedy(g, T, O, O, NM_BF16, 4, 8, vals, m16, nullptr, 0, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(nm_compress(dense, T, O, O, NM_BF16, 3, 4, vals, m16, nullptr, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(mvue_prune_2of4_t(g, T, O, T - 16, NM_BF16, 0, 0, 0, vals, m16, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8(g, T + 16, O, O, NM_BF16, 0, 0, 0, 1.f, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8(g, T, O, O, NM_BF16, 0, 0, 0, -1.f, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8_t(g, T, O, T, NM_BF16, 0, 0, 0, -1.f, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8_t(g, T, O, T - 32, NM_BF16, 0, 0, 0, 1.f, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8_t(g, T + 16, O, T + 16, NM_BF16, 0, 0, 0, 1.f, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8_t(g, T, O, T, NM_BF16, 0, 0, 2, 1.f, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(mvue_prune_1of2_q8_t(g, T, O, T, NM_BF16, 0, 0, 1.f, nullptr, nullptr, m32, nullptr), NM_ERR_NULL);
    EXPECT(mvue_prune_1of2_q8_t(g, T, O, T, NM_BF16, 0, 0, 1.f, nullptr, (uint8_t *)g, m32, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, NM_BF16, 0.5f, ws, wsb, nullptr), NM_ERR_UNSUPPORTED);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, NM_BF16, 0.f, ws, wsb - 1, nullptr), NM_ERR_WORKSPACE);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, NM_BF16, 0.f, nullptr, 0, nullptr), NM_ERR_WORKSPACE);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, NM_BF16, 0.f, (char *)h + 256, wsb, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_update_gemm(vals, m16, h, I, (float *)h, I, T, O, I, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_update_gemm(vals, m16, h, I - 8, dW, I, T, O, I, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, T, O, I, 9, 0.f, ws, wsb, nullptr), NM_ERR_DTYPE);
    EXPECT(nm_update_gemm_q8((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, T, O, I, 1.f, 0.f, (char *)vals + 64, wsb, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_update_gemm_shifted(vals, m16, x0, cb, cb, nullptr, 9, dW, 9 * cb, T, O, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_NULL);
    EXPECT(nm_update_gemm_shifted(vals, m16, x0, cb, cb, shifts, 33, dW, 9 * cb, T, O, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm_shifted(vals, m16, x0, cb, cb, shifts, 9, dW, 9 * cb, T, O, NM_BF16, 0.f, (char *)x0, wsb_conv, nullptr), NM_ERR_ALIAS);
    EXPECT(nm_update_gemm_q8_shifted((const uint8_t *)vals, m32, (const uint8_t *)x0, cb, cb, shifts, 9, dW, 9 * cb, T, O, 1.f, 0.f, (char *)dW,
                                     wsb_conv, nullptr), NM_ERR_ALIAS);
    // the static-scratch entry point: a problem whose split-K scratch exceeds the array
    EXPECT(nm_update_gemm_static(vals, m16, h, 4096, dW, 4096, T, 2048, 4096 / 16 * 2, NM_BF16, 0.f, nullptr), NM_OK);
    // absurd sizes: rejected as shapes, with no overflow in the range arithmetic on the way
    EXPECT(mvue_prune_2of4(g, huge, O, O, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, T, huge, huge, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4(g, T, O, huge, NM_BF16, 0, 0, 0, vals, m16, nullptr, 0, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_4of8_approx(g, huge, huge, huge, NM_F32, 0, 0, vals, m32, dense, huge, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_t(g, huge, O, huge, NM_BF16, 0, 0, 0, vals, m16, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8(g, huge, huge, huge, NM_BF16, 0, 0, 0, 1.f, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(mvue_prune_2of4_q8_t(g, huge, huge, huge, NM_BF16, 0, 0, 0, 1.f, nullptr, (uint8_t *)vals, m32, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_compress(dense, huge, huge, huge, NM_F32, 2, 4, vals, m16, nullptr, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, I, huge, O, I, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm(vals, m16, h, I, dW, huge, T, O, I, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm_q8((const uint8_t *)vals, m32, (const uint8_t *)h, I, dW, I, huge, huge, I, 1.f, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm_shifted(vals, m16, x0, cb, cb, shifts, 9, dW, 9 * cb, huge, O, NM_BF16, 0.f, ws, wsb, nullptr), NM_ERR_SHAPE);
    EXPECT(nm_update_gemm_q8_shifted((const uint8_t *)vals, m32, (const uint8_t *)x0, cb, cb, shifts, 9, dW, huge, T, O, 1.f, 0.f, ws, wsb, nullptr),
           NM_ERR_SHAPE);
    // ---- layers.  Addresses only: nothing is dereferenced on the host
    {
        char *base = (char *)((uintptr_t)1 << 32);
        void *a = base, *b = base + ((int64_t)1 << 40), *out = base + ((int64_t)2 << 40), *bias = base + ((int64_t)3 << 40), *gout = base + ((int64_t)4 << 40),
             *lws = base + ((int64_t)5 << 40);
        const int64_t ld_most = (int64_t)1 << 21, lim = (int64_t)1 << 21;
        auto linear = [&](int64_t T_, int64_t O_, int64_t I_, int m, int mode, int q8, void *act, int64_t ldg, int64_t ldh, void *db, void *w_) {
            return nm_linear_update(a, ldg, act, ldg, b, ldh, T_, O_, I_, m, mode, q8, 1, 2, act ? gout : nullptr, O_, out, db, w_,
                                    nm_linear_update_workspace(T_, O_, I_, q8, db != nullptr), nullptr);
        };
        void *act = base + ((int64_t)6 << 40);
        for (int64_t T_ : {(int64_t)1, (int64_t)77, (int64_t)1024})
            for (int q8 = 0; q8 < 2; ++q8) {
                EXPECT(linear(T_, 64, 128, 4, 0, q8, nullptr, 64, 128, bias, lws), NM_OK);
                EXPECT(linear(T_, 2048, 128, 4, 1, q8, nullptr, 2048, 128, nullptr, lws), NM_OK);
                EXPECT(linear(T_, 64, 128, 2, 0, q8, nullptr, 72, 136, bias, lws), NM_OK);
                EXPECT(linear(T_, 8, 16, 4, 0, q8, nullptr, ld_most, ld_most, bias, lws), NM_OK);
                EXPECT(linear(T_, 8, 16, 4, 0, q8, nullptr, ld_most + 8, 16, bias, lws), NM_ERR_SHAPE);
                EXPECT(linear(T_, 8, 16, 4, 0, q8, nullptr, 8, ld_most + 8, bias, lws), NM_ERR_SHAPE);
            }
        EXPECT(linear(100, 64, 128, 4, 0, 0, act, 64, 128, bias, lws), NM_OK);
        EXPECT(linear(100, 64, 128, 4, 0, 1, act, 64, 128, bias, lws), NM_ERR_UNSUPPORTED);
        EXPECT(linear(100, 64, 128, 3, 0, 0, nullptr, 64, 128, bias, lws), NM_ERR_UNSUPPORTED);
        EXPECT(linear(100, 64, 128, 2, 1, 0, nullptr, 64, 128, bias, lws), NM_ERR_UNSUPPORTED);
        EXPECT(linear(100, 64, 128, 4, 0, 0, nullptr, 64, 128, bias, nullptr), NM_ERR_WORKSPACE);
        EXPECT(linear(100, 64, 128, 4, 0, 0, nullptr, 64, 128, out, lws), NM_ERR_ALIAS);
        EXPECT(linear(100, 64, 128, 4, 0, 0, nullptr, 64, 128, (char *)bias + 2, lws), NM_ERR_ALIGN);
        for (int64_t bad : {(int64_t)0, (int64_t)-16, huge, INT64_MAX, INT64_MIN}) {
            EXPECT(linear(bad, 64, 128, 4, 0, 0, nullptr, 64, 128, bias, lws), NM_ERR_SHAPE);
            EXPECT(linear(100, bad, 128, 4, 0, 0, nullptr, bad, 128, bias, lws), NM_ERR_SHAPE);
            EXPECT(linear(100, 64, bad, 4, 0, 1, nullptr, 64, bad, bias, lws), NM_ERR_SHAPE);
            EXPECT(linear(100, 64, 128, 4, 0, 0, nullptr, bad == huge ? bad : -8, 128, bias, lws), NM_ERR_SHAPE);
            if (nm_linear_update_workspace(bad, 64, 128, 0, 1) || nm_linear_update_workspace(64, bad, 128, 0, 1) || nm_linear_update_workspace(64, 64, bad, 1, 1)) ++failures;
        }
        EXPECT(linear((((int64_t)1 << 34) / lim) + 1, lim, 16, 4, 0, 0, nullptr, lim, 16, bias, lws), NM_ERR_SHAPE);
        if (!nm_linear_update_workspace(((int64_t)1 << 34) / lim, lim, 16, 0, 1) || !nm_linear_update_workspace((int64_t)1 << 31, 8, 32, 1, 1)) ++failures;

        // the dense products: x [T x I] and g [T x O] at a, w at b, y and dx at out
        auto forward = [&](int64_t T_, int64_t O_, int64_t I_, int64_t ldx, const void *x_, const void *bias_, void *y) {
            return nm_linear_forward(x_, ldx, b, bias_, T_, O_, I_, 1, y, nullptr);
        };
        auto input_grad = [&](int64_t T_, int64_t O_, int64_t I_, int64_t ldg, const void *w_, void *dx) { return nm_linear_input_grad(a, ldg, w_, T_, O_, I_, dx, nullptr); };
        for (int64_t T_ : {(int64_t)1, (int64_t)77, (int64_t)1 << 31}) {
            EXPECT(forward(T_, 8, 16, 16, a, bias, out), NM_OK);
            EXPECT(input_grad(T_, 8, 16, 8, b, out), NM_OK);
            const int wide = T_ < 1024 ? NM_OK : NM_ERR_ALIAS;          // (2^31 rows of 4 MB reach over the other tensors)
            EXPECT(forward(T_, 8, 16, ld_most, a, nullptr, out), wide);
            EXPECT(input_grad(T_, 8, 16, ld_most, b, out), wide);
        }
        EXPECT(forward(((int64_t)1 << 34) / lim, lim, 8, 8, a, bias, out), NM_OK);
        EXPECT(forward(((int64_t)1 << 34) / lim + 1, lim, 8, 8, a, bias, out), NM_ERR_SHAPE);
        EXPECT(forward(64, 64, 128, 128, nullptr, bias, out), NM_ERR_NULL);
        EXPECT(forward(64, 64, 128, 128, a, bias, nullptr), NM_ERR_NULL);
        EXPECT(forward(64, 64, 128, 132, a, bias, out), NM_ERR_ALIGN);
        EXPECT(forward(64, 64, 128, 128, (char *)a + 8, bias, out), NM_ERR_ALIGN);
        EXPECT(forward(64, 64, 128, 128, a, (char *)bias + 2, out), NM_ERR_ALIGN);
        EXPECT(forward(64, 64, 128, 128, a, bias, (char *)out + 4), NM_ERR_ALIGN);
        EXPECT(forward(64, 64, 128, 128, a, bias, (char *)a + 64 * 128 * 2 - 16), NM_ERR_ALIAS);
        EXPECT(forward(64, 64, 128, 128, a, bias, (char *)b + 64 * 128 * 2 - 16), NM_ERR_ALIAS);
        EXPECT(forward(64, 64, 128, 128, a, (char *)out + 64 * 64 * 2 - 16, out), NM_ERR_ALIAS);
        EXPECT(forward(64, 64, 128, 128, a, bias, (char *)a + 64 * 128 * 2), NM_OK);
        EXPECT(input_grad(64, 64, 128, 64, nullptr, out), NM_ERR_NULL);
        EXPECT(input_grad(64, 64, 128, 68, b, out), NM_ERR_ALIGN);
        EXPECT(input_grad(64, 64, 128, 64, (char *)b + 2, out), NM_ERR_ALIGN);
        EXPECT(input_grad(64, 64, 128, 64, b, (char *)a + 64 * 64 * 2 - 16), NM_ERR_ALIAS);
        EXPECT(input_grad(64, 64, 128, 64, b, (char *)b - 64 * 128 * 2 + 16), NM_ERR_ALIAS);
        for (int64_t bad : {(int64_t)0, (int64_t)-16, huge, INT64_MAX, INT64_MIN}) {
            EXPECT(forward(bad, 64, 128, 128, a, bias, out), NM_ERR_SHAPE);
            EXPECT(forward(64, bad, 128, 128, a, bias, out), NM_ERR_SHAPE);
            EXPECT(forward(64, 64, bad, bad, a, bias, out), NM_ERR_SHAPE);
            EXPECT(forward(64, 64, 128, bad, a, bias, out), NM_ERR_SHAPE);
            EXPECT(input_grad(64, bad, 128, bad, b, out), NM_ERR_SHAPE);
            EXPECT(input_grad(64, 64, 128, bad, b, out), NM_ERR_SHAPE);
        }
        EXPECT(forward(64, 60, 128, 128, a, bias, out), NM_ERR_SHAPE);
        EXPECT(input_grad(64, 64, 100, 64, b, out), NM_ERR_SHAPE);

        auto conv = [&](int64_t N, int64_t C, int64_t O_, int64_t H, int64_t W, int k, int q8, int mode, const void *x_, void *dW_, void *w_) {
            return nm_conv_update(a, 0, x_, 1, N, C, O_, H, W, k, q8, mode, 1, 2, dW_, w_, nm_conv_update_workspace(N, C, O_, H, W, k, q8), nullptr);
        };
        for (int q8 = 0; q8 < 2; ++q8)
            for (int mode = 0; mode < 2; ++mode)
                for (int k : {1, 3, 5}) {
                    EXPECT(conv(2, 64, 64, 14, 14, k, q8, mode, b, out, lws), NM_OK);
                    EXPECT(conv(1, 16, 8, 1, 300, k, q8, mode, b, out, lws), NM_OK);
                }
        // kernel sizes whose square does not fit an int among them
        for (int k : {0, -1, -3, 2, 4, 7, 9, 46339, 46341, 65535, 65537, INT32_MAX, INT32_MIN, INT32_MIN + 1}) {
            EXPECT(conv(2, 64, 64, 14, 14, k, 0, 0, b, out, lws), NM_ERR_SHAPE);
            if (nm_conv_update_workspace(2, 64, 64, 14, 14, k, 1)) ++failures;
        }
        for (int64_t bad : {(int64_t)0, (int64_t)-8, ((int64_t)1 << 20) + 16, huge, INT64_MAX, INT64_MIN}) {
            EXPECT(conv(bad, 64, 64, 14, 14, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
            EXPECT(conv(2, bad, 64, 14, 14, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
            EXPECT(conv(2, 64, bad, 14, 14, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
            EXPECT(conv(2, 64, 64, bad, 14, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
            EXPECT(conv(2, 64, 64, 14, bad, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
        }
        EXPECT(conv(1 << 20, 8, 8, 1 << 20, 1 << 10, 5, 0, 0, b, out, lws), NM_ERR_SHAPE);
        EXPECT(conv(2, 1 << 20, 8, 14, 1 << 20, 5, 0, 0, b, out, lws), NM_ERR_SHAPE);
        EXPECT(conv(2, 24, 64, 14, 14, 3, 1, 0, b, out, lws), NM_ERR_SHAPE);
        EXPECT(conv(2, 64, 60, 14, 14, 3, 0, 0, b, out, lws), NM_ERR_SHAPE);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 2, b, out, lws), NM_ERR_UNSUPPORTED);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, nullptr, out, lws), NM_ERR_NULL);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, nullptr, lws), NM_ERR_NULL);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, (char *)b + 8, out, lws), NM_ERR_ALIGN);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, (char *)out + 2, lws), NM_ERR_ALIGN);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, out, nullptr), NM_ERR_WORKSPACE);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, (char *)b + 64, lws), NM_ERR_ALIAS);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, out, (char *)a - 256), NM_ERR_ALIAS);
        EXPECT(conv(2, 64, 64, 14, 14, 3, 0, 0, b, out, (char *)out + 256), NM_ERR_ALIAS);
        EXPECT(nm_conv_update(a, 0, b, 0, 2, 64, 64, 14, 14, 3, 0, 0, 1, 2, out, lws, nm_conv_update_workspace(2, 64, 64, 14, 14, 3, 0) - 1, nullptr),
               NM_ERR_WORKSPACE);
    }
    if (failures) { fprintf(stderr, "abi sanitizer driver: %d failures\n", failures); return 1; }
    printf("abi sanitizer driver ok (%d stub launches)\n", g_launches);
    return 0;
}
