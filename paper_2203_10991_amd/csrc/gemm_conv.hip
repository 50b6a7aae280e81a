// Update GEMM of a 3 x 3 convolution, all nine taps of a channel block in one workgroup:
//     part[slab][o][tap][c] = sum over the slab's tokens t of theta(g)[t][o] * x[t + shift(tap)][c]
// on the zero-padded channels-last grid (conv_grid.hip).  The nine taps read the SAME rows of x, shifted: a general tile kernel
// on shifted views (update_gemm_smfmac_kernel<..., SHIFTED>) fetches every row once per tap and is bound by that path from the
// L2s (17 TB/s of the 87 us it took on ResNet-50's first 3x3 stage).  Here the rows sit once in a ring in LDS and the taps are
// read from it at their shifts, so a 64 x 9*CB tile of dW fetches 1/9 of the bytes of x per product.
//
// Workgroup = 12 waves (three per SIMD): 64 rows of dW x 9*CB columns (CB = 64 or 32 channels), every wave 2 x 3 accumulator blocks
// of 32 x 32 (96 registers).  9*CB columns are NWN = 6 or 3 waves wide; the other factor of 12 splits the tokens: KG = 2 or 4 groups
// of waves each take one MFMA step (32 tokens, 64 with 8-bit operands) of a super-stage of KG steps and are summed through LDS at
// the end, in a fixed order.
//
// LDS: [0, 64 KB) ring of x rows, CB channels each; 8 blocks of 8 KB, a super-stage's rows per block.  A super-stage s reads the blocks
// s .. s+P, P = ceil(2 * margin / rows per block).  The ring is addressed with 16-bit adds, which wrap by themselves.
// Then 8 slots of vals fragments and index words, one per super-stage.  During super-stage s: the operands of s are in registers,
// those of s+1 have landed in LDS and replace them register by register behind the last MFMA that reads them, the loads of s+2
// and s+3 are in flight and those of s+4 are issued.  Bank conflicts of the transposing reads (four, or with 8-bit operands
// eight, consecutive rows at any shift): rows of 32 channels need nothing (four resp. eight of them are 256 contiguous bytes);
// with 64 channels the halves of a row are exchanged by bit 1 (bit 2) of the row number.
//
// Bound: matrix pipeline at the clock the power limit leaves (59 % busy at 1.7 GHz on a long 14 x 14 layer, no bank conflicts, LDS
// 40 % busy); what it waits for is the barrier per super-stage of 576 matrix cycles, so the loads' address arithmetic between the
// barriers was cut to two multiplies (with descriptors rebuilt per load: 166 instead of 150 us there).  On grids with few
// channels one pass over x and the compressed gradient.  Measured at batch 256, general kernel -> this one: 56 x 56 x 64
// 87 -> 42 us (8-bit 47 -> 43), 14 x 14 x 256 60 -> 51 us (8-bit
// 38 -> 31), 7 x 7 x 512 70 -> 58 us (8-bit 51 -> 34).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "nm_internal.h"
#include "smfmac_common.h"

namespace nm {

constexpr int CG_WAVES = 12, CG_TM = 64, CG_AHEAD = 4;               // CG_AHEAD: super-stages the loads run ahead
constexpr int CG_RING = 65536, CG_BLOCK = 8192, CG_SLOTS = 8;
constexpr int CG_XCH = 6 * 6 * 64 * 64;                              // bytes of accumulators exchanged at a time: six waves' blocks

template <bool Q8, int CB> struct ConvTile {
    static constexpr int ESZ = Q8 ? 1 : 2;
    static constexpr int NWN = 9 * CB / 96, KG = CG_WAVES / NWN;      // waves across the columns; token groups of waves
    static constexpr int STEP = Q8 ? 64 : 32;                         // tokens of an MFMA step
    static constexpr int SS = STEP * KG;                              // tokens of a super-stage
    static constexpr int RB = CB * ESZ;                               // bytes of a ring row
    static constexpr int MW = Q8 ? 4 : 2, MB = 256;                   // bytes of an index word; of a token group's in LDS (one load of 64 lanes)
    static constexpr int SLOT = 2 * KG * (CG_TM * 16 + MB);           // vals and index words of a super-stage
    static constexpr int LDS = CG_RING + CG_SLOTS * SLOT > CG_XCH ? CG_RING + CG_SLOTS * SLOT : CG_XCH;
    static_assert(SS * RB == CG_BLOCK && LDS <= 160 * 1024, "ring blocks");
};

union ConvB { bf16x16 v16; i32x8 v8; u32x2 q[4]; s16x4 h[4]; };
union ConvI { u32x2 w2; uint32_t w[2]; };
union ConvA { bf16x8 v16; i32x4 v8; u32x4 u4; };

__device__ __forceinline__ uint32_t add_u16(uint32_t s, uint32_t v)   // (s + v) mod 2^16
{
    uint32_t r;
    asm volatile("v_add_u16 %0, %1, %2" : "=v"(r) : "s"(s), "v"(v));
    return r;
}

template <bool Q8, int CB>
__global__ __launch_bounds__(CG_WAVES * 64) void conv_gemm_kernel(
    const char *__restrict__ vals, const char *__restrict__ meta, const char *__restrict__ x,      // x: row -margin of the grid; T + P*SS rows
    float *__restrict__ part, int64_t T, int ss_per_slab, int O, int C, int tiles_n, int margin, ShiftArg sh)
{
    using Tile = ConvTile<Q8, CB>;
    constexpr int ESZ = Tile::ESZ, NWN = Tile::NWN, KG = Tile::KG, STEP = Tile::STEP, SS = Tile::SS, RB = Tile::RB, MB = Tile::MB;
    constexpr int GPS = 2 * KG;                                       // token groups of a super-stage
    // (the kernel's only LDS object: the ring starts at address 0, which its 16-bit addresses assume)
    __shared__ __attribute__((aligned(1024))) char S[Tile::LDS];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % NWN, kgrp = wave / NWN;
    // consecutive workgroups of an XCD take tiles of one slab: they share its rows of x and vals through the L2
    const unsigned n = gridDim.x, xcd = blockIdx.x % 8, first = xcd * (n / 8) + min(xcd, n % 8), w_id = first + blockIdx.x / 8;
    const int tiles = ((O + CG_TM - 1) / CG_TM) * tiles_n;
    const int slab = (int)(w_id / tiles), tile = (int)(w_id % tiles);
    const int o0 = (tile / tiles_n) * CG_TM, c0 = (tile % tiles_n) * CB;
    const int64_t n_ss_all = T / SS, ss0 = (int64_t)slab * ss_per_slab;
    const int n_ss = (int)min((int64_t)ss_per_slab, n_ss_all - ss0);
    const int P = (2 * margin + SS - 1) / SS;

    f32x16 acc[2][3];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc_zero<true>(acc[a][b]);

    // ---- direct loads: waves 0-3 bring two kilobytes of an x block each, waves 4 .. 4+GPS-1 one token group's vals and index
    // words.  Every wave with a part issues two loads per super-stage, which is what the waits count.  A wave's addresses are
    // two descriptors at the slab's start, a lane offset, and a scalar offset that advances by a super-stage and stops at the
    // tensor's last one: what is loaded again there is not used.  (Every scalar instruction here delays the next barrier.)
    const int64_t xrow = (int64_t)C * ESZ, G0 = ss0 * GPS + (wave - 4);
    const char *base0 = wave < 4 ? x + ss0 * SS * xrow : vals + G0 * O * 16, *base1 = wave < 4 ? base0 : meta + G0 * O * Tile::MW;
    const __amdgpu_buffer_rsrc_t r0 = __builtin_amdgcn_make_buffer_rsrc((void *)base0, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc((void *)base1, 0, 0x7fffffff, 0x00020000);
    const uint32_t step0 = wave < 4 ? (uint32_t)(SS * xrow) : (uint32_t)(GPS * O * 16), step1 = wave < 4 ? step0 : (uint32_t)(GPS * O * Tile::MW);
    uint32_t src[2], lds[2], lds_step = wave < 4 ? CG_BLOCK : Tile::SLOT;
    if (wave < 4) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int at = (2 * wave + i) * 1024 + lane * 16, r = at / RB;
            int pos = (at % RB) / 16;
            if constexpr (CB == 64) pos ^= ((r >> (Q8 ? 2 : 1)) & 1) * (RB / 32);
            src[i] = (uint32_t)(r * xrow + c0 * ESZ + pos * 16);
            lds[i] = (uint32_t)(2 * wave + i) * 1024;
        }
    } else {
        src[0] = (uint32_t)min(o0 + 2 * (lane & 31) + (lane >> 5), O - 1) * 16u;       // slot q holds row 2*(q%32) + q/32
        src[1] = Q8 ? (uint32_t)min(o0 + lane, O - 1) * 4u : (uint32_t)min(o0 + 2 * (lane & 31), O - 2) * 2u;
        lds[0] = (uint32_t)(CG_RING + (wave - 4) * (CG_TM * 16));
        lds[1] = (uint32_t)(CG_RING + GPS * (CG_TM * 16) + (wave - 4) * MB);
    }
    const int loader = wave < 4 ? 1 : wave < 4 + GPS ? 2 : 0;
    const int last = (int)min((int64_t)0x7fffffff, n_ss_all - 1 - ss0) + (wave < 4 ? P : 0);      // last block (super-stage) there is
    // block (waves 0-3) or super-stage `i` of the slab
    auto load_at = [&](int i) {
        const uint32_t from = (uint32_t)min(i, last), to = (uint32_t)(i & 7) * lds_step;
        if (loader == 1) {
            load16_to_lds(r0, S + lds[0] + to, src[0], from * step0);
            load16_to_lds(r0, S + lds[1] + to, src[1], from * step0);
        } else if (loader == 2) {
            load16_to_lds(r0, S + lds[0] + to, src[0], from * step0);
            load4_to_lds(r1, S + lds[1] + to, src[1], from * step1);
        }
    };
    const int ahead = wave < 4 ? P : 0;
    auto load_stage = [&](int s) { load_at(s + ahead); };             // what super-stage s needs beyond its predecessors

    // ---- LDS reads.  bf16: read j of a B fragment covers 4 tokens at +4*(j%2) + 16*(j/2), 8-bit: 8 tokens at +8*(j%2) + 32*(j/2)
    const int li = lane & 15, hi = lane >> 5, grp = (lane >> 4) & 1;
    uint32_t b_at[3];                                                 // ring address of the lane's first read in super-stage 0
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int blk = 3 * wn + b, tap = blk / (CB / 32), half = blk % (CB / 32);
        const int row = kgrp * STEP + sh.rows[tap] + margin + (Q8 ? 16 * hi + (li >> 1) : 8 * hi + (li >> 2));
        const int in_row = Q8 ? grp * 16 + (li & 1) * 8 : (2 * grp + ((li & 3) >> 1)) * 16 + (li & 1) * 8;
        const int h = CB == 64 ? half ^ ((row >> (Q8 ? 2 : 1)) & 1) : 0;
        b_at[b] = (uint32_t)(row * RB + h * (RB / 2) + in_row);
    }
    const uint32_t a_at = (uint32_t)(CG_RING + (2 * kgrp + hi) * (CG_TM * 16) + (lane & 31) * 16);
    const uint32_t m_at = (uint32_t)(CG_RING + GPS * (CG_TM * 16) + (2 * kgrp + hi) * MB + (lane & 31) * (2 * Tile::MW));
    // the sparse operand's fragments and index words in two sets, the dense operand's in one that is refilled in place
    ConvA af[2][2];
    ConvB bf[3];
    ConvI ix[2];
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        ix[set].w2 = u32x2{0, 0};
#pragma unroll
        for (int a = 0; a < 2; ++a) af[set][a].u4 = u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) bf[b].q[j] = u32x2{0, 0};
    auto read_b = [&](auto b_c, int s) {
        constexpr int b = decltype(b_c)::value, D1 = (Q8 ? 8 : 4) * RB, D2 = (Q8 ? 32 : 16) * RB;
        const uint32_t so = (uint32_t)(s & 7) * CG_BLOCK;
        const uint32_t p0 = add_u16(so, b_at[b]), p1 = add_u16(so + D1, b_at[b]), p2 = add_u16(so + D2, b_at[b]), p3 = add_u16(so + D1 + D2, b_at[b]);
        if constexpr (Q8) {
            lds_refill_tr8<0>(bf[b].q[0], p0);
            lds_refill_tr8<0>(bf[b].q[1], p1);
            lds_refill_tr8<0>(bf[b].q[2], p2);
            lds_refill_tr8<0>(bf[b].q[3], p3);
        } else {
            lds_refill_tr16<0>(bf[b].h[0], p0); lds_refill_tr16<0>(bf[b].h[1], p1);
            lds_refill_tr16<0>(bf[b].h[2], p2); lds_refill_tr16<0>(bf[b].h[3], p3);
        }
    };
    auto read_a = [&](auto set_c, int s) {                            // three reads
        constexpr int set = decltype(set_c)::value;
        const uint32_t so = (uint32_t)(s & 7) * Tile::SLOT;
        lds_refill_b128<0>(af[set][0].u4, a_at + so);
        lds_refill_b128<512>(af[set][1].u4, a_at + so);
        if constexpr (Q8) lds_refill_b64<0>(ix[set].w2, m_at + so);
        else lds_refill_b32<0>(ix[set].w[0], m_at + so);
    };
    auto mfma2 = [&](auto set_c, auto b_c) {                          // column block b against both row blocks
        constexpr int set = decltype(set_c)::value, b = decltype(b_c)::value;
        if constexpr (Q8) {
            smfmac_32x32x64_bf8_fp8<true>(acc[0][b], af[set][0].v8, bf[b].v8, ix[set].w[0]);
            smfmac_32x32x64_bf8_fp8<true>(acc[1][b], af[set][1].v8, bf[b].v8, ix[set].w[1]);
        } else {
            smfmac_32x32x32<-1, 0, true>(acc[0][b], af[set][0].v16, bf[b].v16, ix[set].w[0]);
            smfmac_32x32x32<-1, 1, true>(acc[1][b], af[set][1].v16, bf[b].v16, ix[set].w[0]);
        }
    };
    using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>; using I2 = std::integral_constant<int, 2>;

    // ---- prologue: the blocks before the first super-stage's own, then CG_AHEAD super-stages
    if (wave < 4)
        for (int b = 0; b < P; ++b) load_at(b);
    for (int s = 0; s < CG_AHEAD; ++s) load_stage(s);
    wait_vmcnt<2 * (CG_AHEAD - 1)>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // Super-stage s.  Reads in flight when it starts, in order: its B0 B1 B2, four each; with the three of the next sparse
    // fragments and the refills behind them, 11 are always younger than the four that the next MFMAs wait for.
    auto super_stage = [&](auto set_c, int s) {
        constexpr int set = decltype(set_c)::value;
        // super-stage s+1 has landed, everywhere; every wave is past the reads of s-1, whose ring block and slot the loads take
        wait_vmcnt<2 * (CG_AHEAD - 2)>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        read_a(std::integral_constant<int, 1 - set>{}, s + 1);
        asm volatile("s_waitcnt lgkmcnt(11)" ::: "memory");
        mfma2(set_c, I0{});
        read_b(I0{}, s + 1);
        load_stage(s + CG_AHEAD);
        asm volatile("s_waitcnt lgkmcnt(11)" ::: "memory");
        mfma2(set_c, I1{});
        read_b(I1{}, s + 1);
        asm volatile("s_waitcnt lgkmcnt(11)" ::: "memory");
        mfma2(set_c, I2{});
        read_b(I2{}, s + 1);
    };
    read_a(I0{}, 0);
    read_b(I0{}, 0); read_b(I1{}, 0); read_b(I2{}, 0);
    for (int s = 0; s < n_ss; s += 2) {
        super_stage(I0{}, s);
        if (s + 1 < n_ss) super_stage(I1{}, s + 1);
    }
    // the matrix pipeline may still write the last accumulators; loads and reads that ran ahead must not land in the exchange
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    // (the fragments are not used any more, but their registers are theirs until here: a read that ran ahead writes to them)
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        asm volatile("" : : "v"(ix[set].w2));
#pragma unroll
        for (int a = 0; a < 2; ++a) asm volatile("" : : "v"(af[set][a].u4));
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : : "v"(bf[b].q[j]));
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc_settled<true>(acc[a][b]);
    __syncthreads();

    // ---- the token groups' accumulators are summed through LDS: group g += group g + half, half = KG/2 .. 1
    f32x4 *xch = (f32x4 *)S;
#pragma unroll
    for (int half = KG / 2; half >= 1; half /= 2) {
        if (kgrp >= half && kgrp < 2 * half) {
            f32x4 *dst = xch + (size_t)((kgrp - half) * NWN + wn) * 6 * 4 * 64 + lane;
#pragma unroll
            for (int k = 0; k < 24; ++k) {
                const f32x16 &v = acc[k / 12][(k / 4) % 3];
                dst[k * 64] = f32x4{v[4 * (k % 4)], v[4 * (k % 4) + 1], v[4 * (k % 4) + 2], v[4 * (k % 4) + 3]};
            }
        }
        __syncthreads();
        if (kgrp < half) {
            const f32x4 *from = xch + (size_t)(kgrp * NWN + wn) * 6 * 4 * 64 + lane;
#pragma unroll
            for (int k = 0; k < 24; ++k) {
                const f32x4 v = from[k * 64];
                f32x16 &d = acc[k / 12][(k / 4) % 3];
#pragma unroll
                for (int r = 0; r < 4; ++r) d[4 * (k % 4) + r] += v[r];
            }
        }
        __syncthreads();
    }
    if (kgrp != 0) return;
    const int64_t I = 9 * (int64_t)C;
    float *out = part + (int64_t)slab * O * I;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int blk = 3 * wn + b, tap = blk / (CB / 32), half = blk % (CB / 32);
        const int64_t col = (int64_t)tap * C + c0 + 32 * half + (lane & 31);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = o0 + 2 * (8 * (r >> 2) + 4 * hi + (r & 3)) + a;       // block a holds rows 2m + a
                if (row < O) out[row * I + col] = acc[a][b][r];
            }
    }
}

static int conv_cb(const ConvShape &cs) { return cs.C % 64 == 0 ? 64 : 32; }

// Slabs: enough to give every CU a workgroup, fewer where the partial sums cost more than the shorter slabs save (0.35 us
// per super-stage; partial sums written and read back at about 2.2 MB per us)
static int64_t conv_slabs(const ConvShape &cs, int64_t n_ss)
{
    const int64_t tiles = (int64_t)((cs.O + CG_TM - 1) / CG_TM) * (cs.C / conv_cb(cs));
    const double best = std::sqrt((double)n_ss * 0.35 / ((double)cs.O * cs.C * 36.0 / 2.2e6));
    const int64_t slabs = std::max<int64_t>(1, std::min<int64_t>({256 / tiles, n_ss, (int64_t)(best + 0.5)}));
    const int64_t per = (n_ss + slabs - 1) / slabs;
    return (n_ss + per - 1) / per;
}

// False: not a case of this kernel (another tap count, channels that are no multiple of 32, few of a tile's 64 output channels
// used, an image so wide that the rows between the first and the last tap do not fit the ring beside the blocks in flight, a
// slab beyond what a 31-bit byte offset reaches).
bool conv_gemm_plan(const ConvShape &cs, bool q8, ConvGemmPlan &p)
{
    if (cs.k != 3 || cs.C % 32 || 4 * (int64_t)cs.O < 3 * ((cs.O + CG_TM - 1) / CG_TM * CG_TM)) return false;
    const int64_t ss = CG_BLOCK / (conv_cb(cs) * (q8 ? 1 : 2)), before = (2 * (cs.W + 3) + ss - 1) / ss;
    if (before + CG_AHEAD > 7) return false;
    const int64_t n_ss = ((int64_t)cs.N * (cs.H + 2) * (cs.W + 2) + ss - 1) / ss;
    p.T = n_ss * ss;
    p.x_rows = (n_ss + before) * ss;
    p.slabs = (int)conv_slabs(cs, n_ss);
    const int64_t per = (n_ss + p.slabs - 1) / p.slabs;
    return (per + before + CG_AHEAD) * ss * std::max(cs.C * (q8 ? 1 : 2), cs.O * (q8 ? 1 : 2)) < ((int64_t)1 << 31) - 65536;
}

// x_full: p.x_rows rows of the grid from row -(W+3) on; part: [p.slabs][O][9][C] binary32
hipError_t launch_conv_gemm(const ConvShape &cs, bool q8, const ConvGemmPlan &p, const void *vals, const void *meta, const void *x_full,
                            float *part, hipStream_t st)
{
    const int cb = conv_cb(cs), slabs = p.slabs, tiles_n = cs.C / cb, Wp = cs.W + 2, margin = Wp + 1;
    const int64_t n_ss = p.T / (CG_BLOCK / (cb * (q8 ? 1 : 2)));
    ShiftArg sh{};
    for (int t = 0; t < 9; ++t) sh.rows[t] = (t / 3 - 1) * Wp + (t % 3 - 1);
    const int64_t wgs = (int64_t)((cs.O + CG_TM - 1) / CG_TM) * tiles_n * slabs;
    if (wgs > 0x7fffffffll) return hipErrorInvalidConfiguration;
#define NM_CONV(Q8, CB)                                                                                                                       \
    hipLaunchKernelGGL((conv_gemm_kernel<Q8, CB>), dim3((unsigned)wgs), dim3(CG_WAVES * 64), 0, st, (const char *)vals, (const char *)meta, \
                       (const char *)x_full, part, p.T, (int)((n_ss + slabs - 1) / slabs), cs.O, cs.C, tiles_n, margin, sh)
    if (q8) { if (cb == 64) NM_CONV(true, 64); else NM_CONV(true, 32); }
    else { if (cb == 64) NM_CONV(false, 64); else NM_CONV(false, 32); }
#undef NM_CONV
    return hipGetLastError();
}

}  // namespace nm
