// Update GEMM (eq. (3)) for binary32 operands on the SPARSE 16-bit matrix path.
//
// gfx950 has no sparse (and no fast) binary32 matrix instruction: the dense fp32 MFMA path executes every product at
// 157 TFLOP/s.  Here each binary32 value x is written as a sum of three bf16 terms,
//     x0 = bf16(x),  x1 = bf16(x - x0),  x2 = bf16(x - x0 - x1)          (round to nearest even; both differences are
// exact in binary32), which carries 24 significant bits, and the product of the compressed operand a and the
// activations b is formed from the six partial products whose terms have i + j <= 2:
//     a b ~ a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0).
// The three dropped products are below 2^-24 |a b|.  One launch writes the three planes of both operands (split3_kernel), one GEMM
// holds a stage of all six in LDS and forms the six products from them (update_gemm_x3_kernel): each plane is fetched once, where a
// 16-bit GEMM over stacked planes fetched the leading ones three times.  The product of the leading terms has accumulators of
// its own and the five others theirs, added at the end: small terms are never rounded against large sums.
//
// Non-finite inputs: the first plane carries the infinity or NaN, the other two are zero; the results they touch are
// non-finite, though an infinity may come out as a NaN (infinity times a zero low-order term).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "nm_internal.h"
#include "smfmac_common.h"
#include "gemm_plan.h"

namespace nm {

namespace {

__device__ __forceinline__ uint32_t bf16_rne_bits(float x)          // finite or not: NaN stays NaN (quiet bit kept)
{
    const uint32_t b = __float_as_uint(x);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (b >> 16) | 0x40u;
    return (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ void split3(float x, uint32_t &p0, uint32_t &p1, uint32_t &p2)
{
    p0 = bf16_rne_bits(x);
    const float x0 = __uint_as_float(p0 << 16);
    const bool finite = (__float_as_uint(x0) & 0x7f800000u) != 0x7f800000u;
    const float r1 = finite ? x - x0 : 0.f;
    p1 = bf16_rne_bits(r1);
    const float r2 = r1 - __uint_as_float(p1 << 16);
    p2 = bf16_rne_bits(r2);
}

// rows x cols binary32 (row stride ld) -> stages of `per_stage` rows, three planes of bf16 each: out[stage][plane][row][col]; rows past `rows`, up to
// out_rows, are zeros.  A piece is eight values of a row (cols % 8 == 0).  Bound: HBM, 10 bytes a value.
struct SplitArg { const float *x; int64_t rows, cols, ld, out_rows; int per_stage; uint16_t *out; int64_t blocks; };

__global__ __launch_bounds__(256) void split3_kernel(SplitArg a, SplitArg b)       // the first a.blocks workgroups: a, the others: b
{
    const bool second = (int64_t)blockIdx.x >= a.blocks;
    const SplitArg &s = second ? b : a;
    const int64_t n = ((int64_t)blockIdx.x - (second ? a.blocks : 0)) * 256 + threadIdx.x, per_row = s.cols / 8;
    if (n >= s.out_rows * per_row) return;
    const int64_t r = n / per_row, c = (n - r * per_row) * 8;           // (per_stage: 2 or 32)
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (r < s.rows) {
        const float4 v0 = *(const float4 *)(s.x + r * s.ld + c), v1 = *(const float4 *)(s.x + r * s.ld + c + 4);
        x[0] = v0.x; x[1] = v0.y; x[2] = v0.z; x[3] = v0.w; x[4] = v1.x; x[5] = v1.y; x[6] = v1.z; x[7] = v1.w;
    }
    uint32_t p[3][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) split3(x[j], p[0][j], p[1][j], p[2][j]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        *(uint4 *)(s.out + ((r / s.per_stage * 3 + i) * s.per_stage + r % s.per_stage) * s.cols + c) =
            make_uint4(p[i][0] | (p[i][1] << 16), p[i][2] | (p[i][3] << 16), p[i][4] | (p[i][5] << 16), p[i][6] | (p[i][7] << 16));
}

constexpr int X3_TOKENS = 32;             // of a stage: one MFMA step, two token groups
constexpr int X3_STAGES = 3;              // LDS buffers

// vals: [n_stages][3 planes][2][O][8], h: [n_stages][3 planes][32][I], meta: [n_groups][O] (a last odd group has no index words: its
// kept values are zeros).  out + slab * slab_stride gets the slab's sums.
//
// Workgroup = 2 x 2 waves, one per SIMD with 512 registers, of AB x 2 accumulator blocks in three sets: the leading products of even
// stages, those of odd stages, and the rest.  (Two sets of leading products: each is rounded half as often, which more than makes up for
// the additions at the end.)  Operands of a stage: AB x 3 fragments of the sparse operand, 2 x 3 of the dense one, read from LDS once for
// 12 AB MFMAs.  Rows of a wave are interleaved and the h rows swizzled as in update_gemm_smfmac_kernel, whose LDS image this is, three
// planes of it.
// A stage is two phases: phase 0 multiplies column block 0 while block 1's fragments are read; phase 1 multiplies block 1 while block 0's
// and the sparse operand's fragments of the next stage are read into the registers their last MFMA has freed.  Between the
// phases the next stage has to have landed (one barrier), and the buffer of this one is free: the loads of the stage after the
// next two go there.
//
// Bound: power.  9328 x 2960 x 1976, wide tile, all CUs busy: 73 stages of 1536 matrix cycles take 146k cycles at 1.49 GHz (98 us);
// without the loads 138k at 1.74, without the LDS reads 178k at 2.03 (an earlier order of the loads), MFMAs alone 123k at 2.05 (60 us).  So what counts
// is bytes moved per product: 0.26 KB fetched and 0.5 KB read from LDS an MFMA, against 0.32 and 0.83 of the 384-row kernel over stacked
// planes that did this before (345 -> 300 us; the call 450 -> 366; 2048^3 118 -> 66, 1024^3 59 -> 27, 256 x 512 x 512 34 -> 14).  Eight waves of
// 64 x 64 on the same tile, 0.75 KB from LDS, take the same time within 3 % but have no registers for the second set of leading products.
// Loads in bursts instead of one by one: 180k cycles.  2-norm error against binary64, stacked planes -> now: 256 x 512 x 512 7.3e-8 -> 6.5e-8,
// 2048^3 2.1e-7 -> 1.5e-7, 16384 x 1024 x 1024 3.5e-7 -> 1.7e-7.
template <int AB>
__global__ __launch_bounds__(256) void update_gemm_x3_kernel(
    const uint16_t *__restrict__ vals, const uint16_t *__restrict__ meta, const uint16_t *__restrict__ h, float *__restrict__ out, int64_t ldo,
    int64_t slab_stride, int64_t n_stages, int64_t stages_per_slab, int64_t n_groups, int64_t O, int64_t I, int tiles_m, int tiles_n, int accumulate)
{
    constexpr int WN = 2, NW = 4, WPG = 2, TM = 2 * AB * 32, TN = WN * 64;
    constexpr int CPR = TN / 8, ROWS_PER_DMA = 64 / CPR, B_ROWS = X3_TOKENS / NW, B_DMA = B_ROWS / ROWS_PER_DMA, A_DMA = AB / 2;
    constexpr int H_PLANE = 64 * TN, A_OFF = 3 * H_PLANE, A_PLANE = 2 * TM * 16, M_OFF = A_OFF + 3 * A_PLANE, STAGE = M_OFF + NW * 256;
    constexpr int LPS = 3 * B_DMA + 3 * A_DMA + 1;            // direct loads of a wave and stage
    constexpr bool ODD_IN_VGPR = AB == 4;                     // the odd stages' set: the other two take all 256 accumulation registers
    static_assert(AB == 2 || AB == 4, "index words are read as one or two dwords");
    static_assert(X3_STAGES * STAGE <= 160 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char S[X3_STAGES * STAGE];

    int tm, tn, slab;
    tile_and_slab_of_workgroup(tiles_m, tiles_n, n_stages * X3_TOKENS * 3 * (O + 2 * I), tm, tn, slab);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TN, first = slab * stages_per_slab;
    const int n = (int)min(stages_per_slab, n_stages - first);
    out += slab * slab_stride;

    f32x16 even[AB][2], odd[AB][2], rest[AB][2];
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) { acc_zero(even[a][b]); acc_zero<ODD_IN_VGPR>(odd[a][b]); acc_zero(rest[a][b]); }

    // ---- direct loads.  Rows >= O and columns >= I are clamped to the last ones there are: their products are not stored
    const int wgrp = wave / WPG, wsub = wave % WPG;           // the wave's token group of a stage and its AB * 32 rows of the tile
    uint32_t a_src[A_DMA];
#pragma unroll
    for (int d = 0; d < A_DMA; ++d) {
        const int q = 64 * d + lane;                          // slot q of a wave's rows holds row AB * (q % 32) + q / 32
        a_src[d] = (uint32_t)(wgrp * O + min(m0 + wsub * (AB * 32) + AB * (q % 32) + q / 32, O - 1)) * 16u;
    }
    const uint32_t m_src = (uint32_t)(wgrp * O + min(m0 + wsub * (AB * 32) + 2 * (lane % (AB * 16)), O - 2)) * 2u;
    const int dma_row = lane / CPR, dma_pos = lane % CPR;
    const uint32_t b_src = (uint32_t)(((wave * B_ROWS + dma_row) * I + min(n0 + 8 * (dma_pos ^ (4 * (dma_row & 3))), I - 8)) * 2);
    const uint32_t b_step = (uint32_t)(ROWS_PER_DMA * I * 2), h_plane = (uint32_t)(X3_TOKENS * I * 2), v_plane = (uint32_t)(2 * O * 16);
    // The stage whose loads are being issued: bases of its operands, and their sizes, 0 past the slab's end (then nothing is loaded)
    const char *hp = (const char *)h + first * 3 * h_plane, *vp = (const char *)vals + first * 3 * v_plane, *mp = (const char *)meta + first * 4 * O;
    int64_t m_left = (n_groups - 2 * first) * O * 2;
    int ahead = 0;
    auto next_stage = [&]() {
        hp += 3 * (int64_t)h_plane; vp += 3 * (int64_t)v_plane; mp += 4 * O; m_left -= 4 * O;
        ++ahead;
    };
    // load K of that stage into buffer `buf`
    auto fetch_one = [&](auto k_c, int buf) {
        constexpr int K = decltype(k_c)::value;
        char *stage = S + buf * STAGE;
        auto rsrc = [&](const char *base, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, ahead < n ? (int)bytes : 0, 0x00020000); };
        if constexpr (K < 3 * B_DMA) {
            constexpr int p = K / B_DMA, d = K % B_DMA;
            load16_to_lds(rsrc(hp, 3 * h_plane), stage + p * H_PLANE + (wave * B_ROWS + d * ROWS_PER_DMA) * (TN * 2), b_src + d * b_step, p * h_plane);
        } else if constexpr (K < 3 * B_DMA + 3 * A_DMA) {
            constexpr int p = (K - 3 * B_DMA) / A_DMA, d = (K - 3 * B_DMA) % A_DMA;
            load16_to_lds(rsrc(vp, 3 * v_plane), stage + A_OFF + p * A_PLANE + (wave * A_DMA + d) * 1024, a_src[d], p * v_plane);
        } else {
            load4_to_lds(rsrc(mp, m_left < 4 * O ? (uint32_t)m_left : (uint32_t)(4 * O)), stage + M_OFF + wave * 256, m_src, 0);
        }
    };

    // ---- LDS reads: addresses in the buffer that is read, which advance by a stage
    const int li = lane & 15, q4 = lane >> 4, kg = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)S;
    const uint32_t rd_a = lds0 + (uint32_t)(A_OFF + (kg * TM + wm * (AB * 32) + (lane & 31)) * 16);
    const uint32_t rd_m = lds0 + (uint32_t)(M_OFF + (kg * WPG + wm) * 256 + (lane & 31) * (AB * 2));
    const uint32_t rd_row = lds0 + (uint32_t)((8 * (q4 >> 1) + (li >> 2)) * (TN * 2) + (2 * (q4 & 1) + ((li & 3) >> 1)) * 16 + (li & 1) * 8);
    const uint32_t rd_b0 = rd_row + 64 * ((wn * 2) ^ (li >> 2)), rd_b1 = rd_row + 64 * ((wn * 2 + 1) ^ (li >> 2));

    Frag8 af[3][AB];                                          // [plane][row block]
    Frag16 bf[2][3];                                          // [column block][plane]
    u32x2 ix[2] = {{0, 0}, {0, 0}};                           // the row blocks' index words, a pair to a dword; of this stage and the next
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
        for (int a = 0; a < AB; ++a) af[p][a].u4 = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j) bf[0][p].q[j] = bf[1][p].q[j] = s16x4{0, 0, 0, 0};
    }
    auto read_ix = [&](auto set_c, uint32_t so) {
        constexpr int set = decltype(set_c)::value;
        if constexpr (AB == 4) lds_refill_b64<0>(ix[set], rd_m + so);
        else { uint32_t w = ix[set][0]; lds_refill_b32<0>(w, rd_m + so); ix[set][0] = w; }
    };
    auto read_a = [&](auto p_c, uint32_t so) {                // AB reads
        constexpr int p = decltype(p_c)::value;
        const uint32_t at = rd_a + so;
        static_for<AB>([&](auto a_c) { constexpr int a = decltype(a_c)::value; lds_refill_b128<p * A_PLANE + 512 * a>(af[p][a].u4, at); });
    };
    auto read_b = [&](auto b_c, auto p_c, uint32_t so) {      // four reads
        constexpr int b = decltype(b_c)::value, p = decltype(p_c)::value, R = TN * 2;
        const uint32_t at = (b ? rd_b1 : rd_b0) + so;
        lds_refill_tr16<p * H_PLANE + 0 * R>(bf[b][p].q[0], at);
        lds_refill_tr16<p * H_PLANE + 4 * R>(bf[b][p].q[1], at);
        lds_refill_tr16<p * H_PLANE + 16 * R>(bf[b][p].q[2], at);
        lds_refill_tr16<p * H_PLANE + 20 * R>(bf[b][p].q[3], at);
    };
    using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>; using I2 = std::integral_constant<int, 2>;
    // The loads of a stage are issued one by one behind MFMAs of two phases, 1 and the 0 that follows: in bursts they fill the CU's
    // vector-memory queue, and a wave that waits for it to take a load feeds its SIMD's matrix pipeline nothing.
    constexpr int NM = 12 * AB, EARLY = (LPS + 1) / 2;        // MFMAs of a stage; loads behind phase 1's half of them
    // plane i of the sparse operand against plane j of column block b, in a stage of parity `set`: product number `nr` of the twelve from phase 1 on
    auto mfma = [&](auto i_c, auto j_c, auto b_c, auto set_c, auto nr_c, int load_buf) {
        constexpr int i = decltype(i_c)::value, j = decltype(j_c)::value, b = decltype(b_c)::value, set = decltype(set_c)::value;
        static_for<AB>([&](auto a_c) {
            constexpr int a = decltype(a_c)::value, at = decltype(nr_c)::value * AB + a;
            if constexpr (i + j > 0) smfmac_32x32x32<-1, (a & 1)>(rest[a][b], af[i][a].v, bf[b][j].v, ix[set][a / 2]);
            else if constexpr (set == 0) smfmac_32x32x32<-1, (a & 1)>(even[a][b], af[i][a].v, bf[b][j].v, ix[set][a / 2]);
            else smfmac_32x32x32<-1, (a & 1), ODD_IN_VGPR>(odd[a][b], af[i][a].v, bf[b][j].v, ix[set][a / 2]);
            static_for<LPS>([&](auto k_c) {
                constexpr int k = decltype(k_c)::value;
                constexpr int behind = k < EARLY ? AB + (5 * AB - 1) * k / EARLY : NM / 2 + (NM / 2 - 1) * (k - EARLY) / (LPS - EARLY);
                if constexpr (behind == at) fetch_one(k_c, load_buf);
            });
        });
    };
    // (the counter of LDS reads on their way goes to 15)
    auto wait_reads = [&](auto n_c) { asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(decltype(n_c)::value < 15 ? decltype(n_c)::value : 15) : "memory"); };
    using std::integral_constant;
#define NM_P(i, j, b, nr, buf) mfma(integral_constant<int, i>{}, integral_constant<int, j>{}, integral_constant<int, b>{}, set_c, integral_constant<int, nr>{}, buf)

    // two stages, and what precedes phase 0 of the third's loads
    static_for<2>([&](auto s_c) {
        static_for<LPS>([&](auto k_c) { fetch_one(k_c, decltype(s_c)::value); });
        next_stage();
    });
    static_for<EARLY>([&](auto k_c) { fetch_one(k_c, 2); });
    wait_vmcnt<LPS + EARLY>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_ix(I0{}, 0);
    read_b(I0{}, I0{}, 0); read_a(I2{}, 0); read_b(I0{}, I1{}, 0); read_a(I1{}, 0); read_b(I0{}, I2{}, 0); read_a(I0{}, 0);
    // stage in buffer `buf`, the next one in `next`; `third` is the buffer of the one after
    auto stage_of = [&](auto set_c, int buf, int next, int third) {
        constexpr int set = decltype(set_c)::value;
        const uint32_t so = (uint32_t)(buf * STAGE), sn = (uint32_t)(next * STAGE);
        // phase 0.  Reads on their way, in order: index words, B00, A2 | B01, A1 | B02, A0; then the twelve of column block 1
        wait_reads(integral_constant<int, 8 + 2 * AB>{});
        NM_P(2, 0, 0, 6, third);
        read_b(I1{}, I0{}, so);
        wait_reads(integral_constant<int, 8 + AB>{});
        NM_P(1, 1, 0, 7, third);
        read_b(I1{}, I1{}, so);
        NM_P(1, 0, 0, 8, third);
        wait_reads(integral_constant<int, 8>{});
        NM_P(0, 2, 0, 9, third);
        read_b(I1{}, I2{}, so);
        NM_P(0, 1, 0, 10, third);
        NM_P(0, 0, 0, 11, third);
        next_stage();
        // the next stage has landed, everywhere, and every wave is past its reads of this one
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(LPS) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        // phase 1.  (Its first MFMAs come before anything else that is issued after the barrier)
        NM_P(2, 0, 1, 0, buf);
        __builtin_amdgcn_sched_barrier(0);
        read_ix(integral_constant<int, 1 - set>{}, sn);
        read_b(I0{}, I0{}, sn);
        read_a(I2{}, sn);
        NM_P(1, 1, 1, 1, buf);
        read_b(I0{}, I1{}, sn);
        NM_P(1, 0, 1, 2, buf);
        read_a(I1{}, sn);
        NM_P(0, 2, 1, 3, buf);
        read_b(I0{}, I2{}, sn);
        NM_P(0, 1, 1, 4, buf);
        NM_P(0, 0, 1, 5, buf);
        read_a(I0{}, sn);
    };
#undef NM_P
    int buf = 0, next = 1, third = 2;
    auto rotate = [&]() { const int t = buf; buf = next; next = third; third = t; };
    for (int s = 0; s < n; s += 2) {
        stage_of(I0{}, buf, next, third);
        rotate();
        if (s + 1 < n) stage_of(I1{}, buf, next, third);
        rotate();
    }
    // what ran ahead has landed, and the matrix pipeline is done with the accumulators, before they are read
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) { acc_settled(even[a][b]); acc_settled<ODD_IN_VGPR>(odd[a][b]); acc_settled(rest[a][b]); }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t col = n0 + wn * 64 + b * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t o = m0 + wm * (AB * 32) + AB * (8 * (r >> 2) + 4 * kg + (r & 3)) + a;       // block a holds rows a, AB+a, ...
                if (o < O && col < I) {
                    float *p = out + o * ldo + col, v = (rest[a][b][r] + odd[a][b][r]) + even[a][b][r];
                    *p = accumulate ? *p + v : v;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
}

inline size_t round256(size_t b) { return (b + 255) / 256 * 256; }

// planes of both operands over whole stages
struct X3Layout { int64_t stages; size_t vals, h, part; };
X3Layout x3_layout(int64_t T, int64_t O, int64_t I)
{
    X3Layout l;
    l.stages = (T + X3_TOKENS - 1) / X3_TOKENS;
    l.vals = 0;
    l.h = round256(3 * (size_t)l.stages * 16 * O * 2);
    l.part = l.h + round256(3 * (size_t)l.stages * X3_TOKENS * I * 2);
    return l;
}

// 256 x 128 tiles (wide) or 128 x 128, and slabs of the token axis, by a cost model: microseconds per stage of a tile by the share of the CUs
// that are busy (the matrix pipes' clock follows the power they draw), fill and drain, and the second pass over the partial sums.
// Against forced plans on 16 sizes from 256 x 64 x 64 to 9328 x 2960 x 1976 its choice is the best or within 3 %, once 6 %.
struct X3Plan { bool wide; int tiles_m, tiles_n, slabs; int64_t per_slab; };
X3Plan x3_plan(int64_t T, int64_t O, int64_t I, size_t workspace)
{
    const X3Layout l = x3_layout(T, O, I);
    const int64_t fit = (int64_t)((workspace - l.part) / ((size_t)O * I * 4)), most = std::max<int64_t>(1, std::min(fit, l.stages / 4));
    X3Plan best{};
    double least = 1e300;
    for (int wide = 0; wide < 2; ++wide) {
        const int64_t tm = (O + (wide ? 255 : 127)) / (wide ? 256 : 128), tn = (I + 127) / 128;
        for (int64_t s = 1; s <= most && tm * tn * (s - 1) < 4 * NM_CUS; ++s) {
            const int64_t per = (l.stages + s - 1) / s, slabs = (l.stages + per - 1) / per, wgs = tm * tn * slabs;
            auto round_us = [&](double fill) { return (double)per * (wide ? 1.0 + 0.3 * fill * fill : 0.55 + 0.17 * fill) + (wide ? 3.0 : 1.0) + 9.0 * fill; };
            const double last = (double)(wgs % NM_CUS) / NM_CUS, cost = (double)(wgs / NM_CUS) * round_us(1.0) + (last > 0.0 ? round_us(last) : 0.0) +
                                (slabs > 1 ? 3.0 + (double)(slabs + 1) * O * I * 4.0 / 4.5e6 : 0.0);
            if (cost < least) { least = cost; best = X3Plan{wide != 0, (int)tm, (int)tn, (int)slabs, per}; }
        }
    }
    return best;
}

}  // namespace

inline size_t segment_bytes(int64_t T, int64_t O, int64_t I)
{
    return round256(6 * (size_t)(T / 2) * O * 2) + round256(6 * (size_t)T * I * 2) + round256(6 * (size_t)(T / 16) * O * 2);
}

// What a GEMM over six stacked planes of each operand takes, which this call first was: callers and the static scratch array see the size they
// always did.  [three planes of vals][three planes of h][partial sums] fit in it, each part on a 256-byte boundary; the plan takes
// no more slabs than do.
size_t update_gemm_f32_split_workspace(int64_t T, int64_t O, int64_t I)
{
    if (T <= 0 || O <= 0 || I <= 0) return 0;
    return segment_bytes(T, O, I) + round256(update_gemm_smfmac_workspace(6 * T, O, I, segment_bytes(T, O, I)));
}

hipError_t launch_update_gemm_f32_split(const void *vals, const uint16_t *meta, const void *h, int64_t ldh, float *dW,
                                        int64_t lddw, int64_t T, int64_t O, int64_t I, float beta, void *workspace,
                                        hipStream_t st)
{
    if (O == 0 || I == 0) return hipSuccess;
    if (T == 0) return launch_update_gemm_smfmac(nullptr, meta, nullptr, I, dW, lddw, 0, O, I, beta, nullptr, st);
    char *w = (char *)workspace;
    const X3Layout l = x3_layout(T, O, I);
    const X3Plan p = x3_plan(T, O, I, update_gemm_f32_split_workspace(T, O, I));
    uint16_t *a = (uint16_t *)(w + l.vals), *b = (uint16_t *)(w + l.h);
    SplitArg sa{(const float *)vals, T / 16, O * 8, O * 8, 2 * l.stages, 2, a, 0}, sb{(const float *)h, T, I, ldh, X3_TOKENS * l.stages, X3_TOKENS, b, 0};
    sa.blocks = (sa.out_rows * (sa.cols / 8) + 255) / 256;
    sb.blocks = (sb.out_rows * (sb.cols / 8) + 255) / 256;
    const int64_t wgs = (int64_t)p.tiles_m * p.tiles_n;
    if (sa.blocks + sb.blocks > 0x7fffffffll || wgs > 0x7fffffffll) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(split3_kernel, dim3((unsigned)(sa.blocks + sb.blocks)), dim3(256), 0, st, sa, sb);
    const OutTarget tg = splitk_target(p.slabs, dW, lddw, w + l.part, O, I, beta != 0.f);
    const dim3 grid((unsigned)wgs, 1, (unsigned)p.slabs);
#define NM_X3(AB)                                                                                                                      \
    hipLaunchKernelGGL(update_gemm_x3_kernel<AB>, grid, dim3(256), 0, st, a, meta, b, tg.out, tg.ldo, tg.slab_stride, l.stages, p.per_slab, \
                       T / 16, O, I, p.tiles_m, p.tiles_n, tg.accumulate)
    if (p.wide) NM_X3(4); else NM_X3(2);
#undef NM_X3
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.slabs > 1) e = launch_splitk_reduce(tg.out, p.slabs, dW, lddw, O, I, beta != 0.f, 1.0f, st);
    return e;
}

}  // namespace nm
