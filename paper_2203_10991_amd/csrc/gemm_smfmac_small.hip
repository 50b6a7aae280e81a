// Update GEMM for small problems: 64 x 64 tiles of dW, the tokens split over the eight waves of a workgroup.
//
// What a small problem takes on the tile kernels is latency: 512 x 512 x 256 is eight 128 x 128 tiles of 16 stages behind a barrier each, and
// with more tokens slabs, whose partial sums cost a second launch (1024^3: 17 us, 3 of them in the loop).  Here a wave takes every
// eighth MFMA step (32 tokens) of its workgroup's tile, brings the step's operands into LDS of its own -- so nothing in the loop waits for
// another wave -- two steps ahead, and the eight waves' sums meet in LDS at the end, in a fixed tree.
// 512 x 512 x 256 9.3 -> 5.6 us, 1024^3 17 -> 7.6.  A wave's step is bound by the way to its operands: 0.5 us alone,
// 0.6-0.7 with all CUs busy, which is why long reductions stay on the large tiles.
//
// LDS of a wave and step: h [32 tokens][64 columns] bf16, chunk c of row k at position c ^ 4 (k / 2 % 2) (a transposing read touches the same 32
// bytes of four consecutive rows, of which every second one shares the banks); then vals [2 groups][64 slots] x 16 bytes, slot q holding tile
// row 2 (q % 32) + q / 32; then the index words of the 64 rows for both groups.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "nm_internal.h"
#include "smfmac_common.h"

namespace nm {

namespace {

constexpr int SM_WAVES = 8, SM_RING = 3, SM_TILE = 64;
constexpr int SM_A = 32 * SM_TILE * 2, SM_M = SM_A + 2 * SM_TILE * 16, SM_STEP = SM_M + 2 * SM_TILE * 2;       // bytes up to and of a step's parts
constexpr int SM_LOADS = 7;                                             // direct loads of a step: 4 h, 2 vals, 1 index words
constexpr int SM_SUMS = SM_WAVES * SM_TILE * SM_TILE * 4;
constexpr int SM_LDS = SM_WAVES * SM_RING * SM_STEP > SM_SUMS ? SM_WAVES * SM_RING * SM_STEP : SM_SUMS;
static_assert(SM_LDS <= 160 * 1024 && SM_STEP % 256 == 0, "LDS");

// The eight waves' blocks are summed in a fixed tree, each sum goes through `scale`, and the tile is stored.  S: SM_SUMS bytes at least
template <typename F>
__device__ __forceinline__ void sum_and_store(f32x16 (&acc)[2][2], char *S, int wave, int64_t m0, int64_t n0, float *out, int64_t ldo, int64_t O, int64_t I,
                                              bool accumulate, F scale)
{
    const int tid = threadIdx.x, lane = tid & 63;
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc_settled(acc[a][b]);
    __syncthreads();                                                    // every wave's ring is done with: the sums go there
    float *sums = (float *)S;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)                                // block a holds rows a, 2 + a, ...
                sums[wave * (SM_TILE * SM_TILE) + (2 * (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) + a) * SM_TILE + b * 32 + (lane & 31)] = acc[a][b][r];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SM_TILE * SM_TILE / 4 / (SM_WAVES * 64); ++k) {
        const int at = (k * SM_WAVES * 64 + tid) * 4, row = at / SM_TILE, col = at % SM_TILE;
        float4 v[SM_WAVES];
#pragma unroll
        for (int w = 0; w < SM_WAVES; ++w) v[w] = *(const float4 *)(sums + w * (SM_TILE * SM_TILE) + at);
#pragma unroll
        for (int d = 1; d < SM_WAVES; d <<= 1)
#pragma unroll
            for (int w = 0; w < SM_WAVES; w += 2 * d) add4(v[w], v[w + d]);
        if (m0 + row < O && n0 + col < I) {
            float4 *p = (float4 *)(out + (m0 + row) * ldo + n0 + col);
            v[0] = make_float4(scale(v[0].x), scale(v[0].y), scale(v[0].z), scale(v[0].w));
            if (accumulate) add4(v[0], *p);
            *p = v[0];
        }
    }
}

// Slab and tile of a workgroup.  Up to eight rows of tiles an XCD (every eighth workgroup) takes a run of all slabs' tiles, a column of tiles after the other, so that
// those which read the same columns of h find them in their L2.  As the tile kernels deal them, in turn unless their number divides by eight, every XCD
// read all of h: 9600 x 184 x 5424 79.7 -> 42.2 us, 20032 x 400 x 576 in four slabs 39.0 -> 24.3, in 8 bits 11968 x 88 x 7536 71.5 -> 40.7 and
// 31648 x 192 x 544 in eight 28.8 -> 17.4; 0.95 of the time in the mean over 2494 plans.  With more rows a run holds part of a column, and is up to 1.11 times slower in
// 8 bits (1056 x 616 x 5120 22.2 -> 24.7).
__device__ __forceinline__ int slab_and_tile(int tiles_m, int tiles_n, int &tm, int &tn)
{
    int slab = (int)blockIdx.z;
    if (tiles_m <= 8) {
        const int n_tiles = tiles_m * tiles_n, id = (int)(blockIdx.z * gridDim.x + blockIdx.x), all = (int)(gridDim.x * gridDim.z), xcd = id % 8;
        const int at = xcd * (all / 8) + min(xcd, all % 8) + id / 8;
        // (at + 0.5 over the divisor, in binary32: exact below 2^20, and there are a few thousand at most; integer divisions cost 0.05 us)
        auto quotient = [](int a, int b) { return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b)); };
        slab = quotient(at, n_tiles);
        tn = quotient(at - slab * n_tiles, tiles_m);
        tm = at - slab * n_tiles - tn * tiles_m;
    } else tile_of_workgroup((int)blockIdx.x, tiles_m, tiles_n, tm, tn);
    tm = __builtin_amdgcn_readfirstlane(tm); tn = __builtin_amdgcn_readfirstlane(tn);
    return __builtin_amdgcn_readfirstlane(slab);
}

// h_rows: rows h has, at most n_groups * 16; the rows past it and a token group past the end count as zeros
__global__ __launch_bounds__(SM_WAVES * 64) void update_gemm_smfmac_small_kernel(const uint16_t *__restrict__ vals, const uint16_t *__restrict__ meta,
                                                                               const uint16_t *__restrict__ h, int64_t ldh, int64_t h_rows, float *__restrict__ out,
                                                                               int64_t ldo, int64_t slab_stride, int64_t n_groups, int64_t groups_per_slab, int64_t O,
                                                                               int64_t I, int tiles_m, int tiles_n, int accumulate)
{
    // this slab's operands and sums: slab * groups_per_slab (even) is below n_groups
    int tm, tn;
    const int slab = slab_and_tile(tiles_m, tiles_n, tm, tn);
    const int64_t g0 = slab * groups_per_slab;
    vals += g0 * O * 8; meta += g0 * O; h += g0 * 16 * ldh; out += slab * slab_stride;
    if (n_groups - g0 > groups_per_slab) { n_groups = groups_per_slab; h_rows = groups_per_slab * 16; }
    else { n_groups -= g0; h_rows -= g0 * 16; }

    __shared__ __attribute__((aligned(1024))) char S[SM_LDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)tm * SM_TILE, n0 = (int64_t)tn * SM_TILE;
    const int steps = (int)((n_groups + 1) / 2), mine = (steps - wave + SM_WAVES - 1) / SM_WAVES;      // steps wave, wave + 8, ...
    const int last_tokens = (int)(h_rows - (int64_t)(steps - 1) * 32);                                // of the last step: 1 .. 32

    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc_zero(acc[a][b]);

    // ---- direct loads; columns and rows past the end are clamped (their sums are not stored), tokens past it sent out of range, which drops
    // them: their h rows and kept values are zeroed when the step has landed
    const int row8 = lane >> 3;
    const uint32_t b_src = (uint32_t)((row8 * ldh + min(n0 + 8 * ((lane & 7) ^ (4 * ((row8 >> 1) & 1))), I - 8)) * 2), b_step = (uint32_t)(8 * ldh * 2);
    const uint32_t a_src = (uint32_t)min(m0 + 2 * (lane & 31) + (lane >> 5), O - 1) * 16u;
    const uint32_t m_src = (uint32_t)((lane >> 5) * O + min(m0 + 2 * (lane & 31), O - 2)) * 2u;
    char *ring = S + wave * SM_RING * SM_STEP;
    const char *hp = (const char *)(h + (int64_t)wave * 32 * ldh), *vp = (const char *)(vals + (int64_t)wave * 2 * O * 8), *mp = (const char *)(meta + (int64_t)wave * 2 * O);
    const int64_t h_step = (int64_t)SM_WAVES * 32 * ldh * 2, v_step = (int64_t)SM_WAVES * 2 * O * 16, m_step = (int64_t)SM_WAVES * 2 * O * 2;
    int ahead = 0;                                                      // this wave's step whose loads are being issued
    auto rsrc = [](const char *base, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000); };
    auto fetch = [&](int slot) {
        char *to = ring + slot * SM_STEP;
        const bool there = ahead < mine;
        const int step = wave + ahead * SM_WAVES, tokens = step == steps - 1 ? last_tokens : 32, groups = step == steps - 1 && n_groups % 2 ? 1 : 2;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            load16_to_lds(rsrc(hp, there ? 0x7fffffffu : 0u), to + d * 1024, 8 * d + row8 < tokens ? b_src + d * b_step : 0xffffffffu, 0);
#pragma unroll
        for (int g = 0; g < 2; ++g) load16_to_lds(rsrc(vp, there && g < groups ? 0x7fffffffu : 0u), to + SM_A + g * 1024, a_src, (uint32_t)(g * O * 16));
        load4_to_lds(rsrc(mp, there ? (uint32_t)(groups * O * 2) : 0u), to + SM_M, m_src, 0);
        hp += h_step; vp += v_step; mp += m_step;
        ++ahead;
    };
    auto clear_tail = [&](char *at) {
        const uint4 z = make_uint4(0, 0, 0, 0);
        for (int d = 0; d < 4; ++d)
            if (8 * d + row8 >= last_tokens) *(uint4 *)(at + d * 1024 + lane * 16) = z;
        if (n_groups % 2) *(uint4 *)(at + SM_A + 1024 + lane * 16) = z;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

    const int li = lane & 15, q4 = lane >> 4, kg = lane >> 5;
    const uint32_t base = (uint32_t)(uintptr_t)(lptr_t)ring;
    const uint32_t rd_a = base + (uint32_t)(SM_A + kg * 1024 + (lane & 31) * 16), rd_m = base + (uint32_t)(SM_M + kg * 128 + (lane & 31) * 4);
    const uint32_t rd_b = base + (uint32_t)((8 * (q4 >> 1) + (li >> 2)) * 128 + ((2 * (q4 & 1) + ((li & 3) >> 1)) ^ (4 * ((li >> 3) & 1))) * 16 + (li & 1) * 8);
    const uint32_t rd_b1 = rd_b ^ 64u;                                  // column block 1: the chunks four on, which is bit 2 of a chunk's position
    for (int s = 0; s < SM_RING; ++s) fetch(s);
    int slot = 0;
    for (int s = 0; s < mine; ++s) {
        wait_vmcnt<(SM_RING - 1) * SM_LOADS>();
        if (wave + s * SM_WAVES == steps - 1 && (last_tokens < 32 || n_groups % 2)) clear_tail(ring + slot * SM_STEP);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t so = (uint32_t)(slot * SM_STEP);
        Frag8 af[2];
        Frag16 bf[2];
        uint32_t ix = lds_read_b32<0>(rd_m + so);
        af[0].u4 = lds_read_b128<0>(rd_a + so);
        af[1].u4 = lds_read_b128<512>(rd_a + so);
        static_for<4>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value, off = (16 * (j >> 1) + 4 * (j & 1)) * 128;
            bf[0].q[j] = lds_read_tr16<off>(rd_b + so);
        });
        static_for<4>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value, off = (16 * (j >> 1) + 4 * (j & 1)) * 128;
            bf[1].q[j] = lds_read_tr16<off>(rd_b1 + so);
        });
        // (the fragments pass through the wait, so that nothing made of them is placed above it)
        wait_for_fragments(af, bf, ix);
        smfmac_32x32x32<-1, 0>(acc[0][0], af[0].v, bf[0].v, ix);
        smfmac_32x32x32<-1, 1>(acc[1][0], af[1].v, bf[0].v, ix);
        smfmac_32x32x32<-1, 0>(acc[0][1], af[0].v, bf[1].v, ix);
        smfmac_32x32x32<-1, 1>(acc[1][1], af[1].v, bf[1].v, ix);
        fetch(slot);
        slot = slot == SM_RING - 1 ? 0 : slot + 1;
    }
    sum_and_store(acc, S, wave, m0, n0, out, ldo, O, I, accumulate != 0, [](float v) { return v; });
}

// The same for 8-bit operands.  A step is 64 tokens: h8 [64 tokens][64 columns] bytes, chunk c (16 columns) of row k at position c ^ 2 (k / 4 % 2) (a transposing
// read touches the same 32 bytes of eight consecutive rows, of which every fourth one shares the banks), vals8 as above, then the index words [2 groups][64 rows].
// The tile kernels take 14 us for anything of up to 384 tokens (six stages and a barrier each, however few are needed):
// 256 x 512 x 512 12.8 -> 5.1, 1024^3 21.2 -> 7.4.  A wave's step is bound by the way to its operands, 0.45 us alone and 0.8-1.15 with all CUs busy.
constexpr int S8_A = 64 * SM_TILE, S8_M = S8_A + 2 * SM_TILE * 16, S8_STEP = S8_M + 2 * SM_TILE * 4, S8_LOADS = 8;       // direct loads of a step: 4 h8, 2 vals8, 2 index words
constexpr int S8_LDS = SM_WAVES * SM_RING * S8_STEP > SM_SUMS ? SM_WAVES * SM_RING * S8_STEP : SM_SUMS;
static_assert(S8_LDS <= 160 * 1024 && S8_STEP % 256 == 0, "LDS");

__global__ __launch_bounds__(SM_WAVES * 64) void update_gemm_q8_small_kernel(const uint8_t *__restrict__ vals, const uint32_t *__restrict__ meta,
                                                                            const uint8_t *__restrict__ h, int64_t ldh, float *__restrict__ out, int64_t ldo,
                                                                            int64_t slab_stride, int64_t n_groups, int64_t groups_per_slab, int64_t O, int64_t I,
                                                                            int tiles_m, int tiles_n, int accumulate, AlphaArg alpha)
{
    int tm, tn;
    const int slab = slab_and_tile(tiles_m, tiles_n, tm, tn);
    const int64_t g0 = slab * groups_per_slab;                          // (even, below n_groups)
    vals += g0 * O * 16; meta += g0 * O; h += g0 * 32 * ldh; out += slab * slab_stride;
    n_groups = min(n_groups - g0, groups_per_slab);

    __shared__ __attribute__((aligned(1024))) char S[S8_LDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)tm * SM_TILE, n0 = (int64_t)tn * SM_TILE;
    const int steps = (int)((n_groups + 1) / 2), mine = (steps - wave + SM_WAVES - 1) / SM_WAVES;      // steps wave, wave + 8, ...

    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc_zero(acc[a][b]);

    // ---- direct loads; columns and rows past the end are clamped (their sums are not stored), a second group past the end is sent out of range, which drops
    // it: its h8 rows and kept values are zeroed when the step has landed (its index words may hold anything)
    const int row16 = lane >> 2;
    const uint32_t b_src = (uint32_t)(row16 * ldh + min(n0 + 16 * ((lane & 3) ^ (2 * ((row16 >> 2) & 1))), I - 16)), b_step = (uint32_t)(16 * ldh);
    const uint32_t a_src = (uint32_t)min(m0 + 2 * (lane & 31) + (lane >> 5), O - 1) * 16u, m_src = (uint32_t)min(m0 + lane, O - 1) * 4u;
    char *ring = S + wave * SM_RING * S8_STEP;
    const char *hp = (const char *)(h + (int64_t)wave * 64 * ldh), *vp = (const char *)(vals + (int64_t)wave * 2 * O * 16), *mp = (const char *)(meta + (int64_t)wave * 2 * O);
    const int64_t h_step = (int64_t)SM_WAVES * 64 * ldh, v_step = (int64_t)SM_WAVES * 2 * O * 16, m_step = (int64_t)SM_WAVES * 2 * O * 4;
    int ahead = 0;                                                      // this wave's step whose loads are being issued
    auto rsrc = [](const char *base, bool there) { return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, there ? 0x7fffffff : 0, 0x00020000); };
    auto fetch = [&](int slot) {
        char *to = ring + slot * S8_STEP;
        const bool there = ahead < mine, both = there && !(wave + ahead * SM_WAVES == steps - 1 && n_groups % 2);
#pragma unroll
        for (int d = 0; d < 4; ++d) load16_to_lds(rsrc(hp, d < 2 ? there : both), to + d * 1024, b_src + d * b_step, 0);
#pragma unroll
        for (int g = 0; g < 2; ++g) load16_to_lds(rsrc(vp, g ? both : there), to + S8_A + g * 1024, a_src, (uint32_t)(g * O * 16));
#pragma unroll
        for (int g = 0; g < 2; ++g) load4_to_lds(rsrc(mp, g ? both : there), to + S8_M + g * 256, m_src, (uint32_t)(g * O * 4));
        hp += h_step; vp += v_step; mp += m_step;
        ++ahead;
    };
    auto clear_second_group = [&](char *at) {
        const uint4 z = make_uint4(0, 0, 0, 0);
        *(uint4 *)(at + 2 * 1024 + lane * 16) = z;
        *(uint4 *)(at + 3 * 1024 + lane * 16) = z;
        *(uint4 *)(at + S8_A + 1024 + lane * 16) = z;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

    const int li = lane & 15, kg = lane >> 5;
    const uint32_t base = (uint32_t)(uintptr_t)(lptr_t)ring;
    const uint32_t rd_a = base + (uint32_t)(S8_A + kg * 1024 + (lane & 31) * 16), rd_m = base + (uint32_t)(S8_M + kg * 256 + (lane & 31) * 8);
    const uint32_t rd_b = base + (uint32_t)((16 * kg + (li >> 1)) * SM_TILE + (((lane >> 4) & 1) ^ (2 * ((li >> 3) & 1))) * 16 + (li & 1) * 8);
    const uint32_t rd_b1 = rd_b ^ 32u;                                  // column block 1: the chunks two on, which is bit 1 of a chunk's position
    for (int s = 0; s < SM_RING; ++s) fetch(s);
    int slot = 0;
    for (int s = 0; s < mine; ++s) {
        wait_vmcnt<(SM_RING - 1) * S8_LOADS>();
        if (wave + s * SM_WAVES == steps - 1 && n_groups % 2) clear_second_group(ring + slot * S8_STEP);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t so = (uint32_t)(slot * S8_STEP);
        FragA8 af[2];
        FragB8 bf[2];
        u32x2 ix = lds_read_b64<0>(rd_m + so);
        af[0].u4 = lds_read_b128<0>(rd_a + so);
        af[1].u4 = lds_read_b128<512>(rd_a + so);
        static_for<4>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value, off = (32 * (j >> 1) + 8 * (j & 1)) * SM_TILE;
            bf[0].q[j] = lds_read_tr8<off>(rd_b + so);
        });
        static_for<4>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value, off = (32 * (j >> 1) + 8 * (j & 1)) * SM_TILE;
            bf[1].q[j] = lds_read_tr8<off>(rd_b1 + so);
        });
        wait_for_fragments(af, bf, ix);
        smfmac_32x32x64_bf8_fp8(acc[0][0], af[0].v, bf[0].v, ix[0]);
        smfmac_32x32x64_bf8_fp8(acc[1][0], af[1].v, bf[0].v, ix[1]);
        smfmac_32x32x64_bf8_fp8(acc[0][1], af[0].v, bf[1].v, ix[0]);
        smfmac_32x32x64_bf8_fp8(acc[1][1], af[1].v, bf[1].v, ix[1]);
        fetch(slot);
        slot = slot == SM_RING - 1 ? 0 : slot + 1;
    }
    const float alpha_v = alpha_of(alpha);
    sum_and_store(acc, S, wave, m0, n0, out, ldo, O, I, accumulate != 0, [&](float v) { return v * alpha_v; });
}

}  // namespace

hipError_t launch_update_gemm_smfmac_small(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, int64_t h_rows, float *out, int64_t ldo,
                                           int64_t slab_stride, int slabs, int64_t groups_per_slab, int64_t T, int64_t O, int64_t I, int accumulate, hipStream_t st)
{
    const int tiles_m = (int)((O + SM_TILE - 1) / SM_TILE), tiles_n = (int)((I + SM_TILE - 1) / SM_TILE);
    hipLaunchKernelGGL(update_gemm_smfmac_small_kernel, dim3((unsigned)(tiles_m * tiles_n), 1, (unsigned)slabs), dim3(SM_WAVES * 64), 0, st, (const uint16_t *)vals, meta,
                       (const uint16_t *)h, ldh, h_rows, out, ldo, slab_stride, T / 16, groups_per_slab, O, I, tiles_m, tiles_n, accumulate);
    return hipGetLastError();
}

hipError_t launch_update_gemm_q8_small(const uint8_t *vals8, const uint32_t *meta32, const uint8_t *h8, int64_t ldh, float *out, int64_t ldo, int64_t slab_stride,
                                       int slabs, int64_t groups_per_slab, int64_t T, int64_t O, int64_t I, int accumulate, const AlphaArg &alpha, hipStream_t st)
{
    const int tiles_m = (int)((O + SM_TILE - 1) / SM_TILE), tiles_n = (int)((I + SM_TILE - 1) / SM_TILE);
    hipLaunchKernelGGL(update_gemm_q8_small_kernel, dim3((unsigned)(tiles_m * tiles_n), 1, (unsigned)slabs), dim3(SM_WAVES * 64), 0, st, vals8, meta32, h8, ldh, out, ldo,
                       slab_stride, T / 32, groups_per_slab, O, I, tiles_m, tiles_n, accumulate, alpha);
    return hipGetLastError();
}

}  // namespace nm
