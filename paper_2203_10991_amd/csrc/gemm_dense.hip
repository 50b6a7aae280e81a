// The dense products of a linear layer on bf16 tensors (T tokens, I inputs, O outputs), on the dense matrix cores:
//     forward         y[T x O]  = x[T x I] W[O x I]^T + b, with or without the ReLU behind it
//     input gradient  dx[T x I] = g[T x O] W[O x I]
// binary32 accumulation, bias and ReLU before the one rounding.
//
// Instruction: v_mfma_f32_32x32x16_bf16.  Both operands have 32 rows or columns (lane % 32) and 16 steps of the reduction axis, eight
// consecutive ones to a lane (8 * (lane / 32) on).  The weights are the first operand, so a lane holds four consecutive features of a
// token and stores them together.
//
// Workgroup = WM x WN waves, each AM x AN blocks of 32 tokens x 32 features.  The reduction axis advances in stages of 64, NS of which rotate
// through LDS, filled by direct loads.  A row that is contiguous along the reduction axis is eight chunks of 16 bytes, chunk c at position
// c ^ (row / 2 % 8), which makes the 16-byte reads of consecutive rows free of bank conflicts; W of the input gradient is contiguous
// along the features instead and is read with ds_read_b64_tr_b16 as the dense operand of the update GEMM is.
// A workgroup takes tiles one after the other, and the stages run on across them: while a tile is converted and stored the next one's first stages
// are on their way (16384 x 1024 -> 4096, four tiles a workgroup: 137 us with a workgroup to a tile and the tile through LDS, now 128).
// A stage is four MFMA steps.  Behind the second the next stage has to have landed (one barrier) and this stage's last fragments are in
// registers, so its buffer is free and the loads of the stage NS later go there; the next stage's first fragments are read under the last two steps.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "nm_internal.h"
#include "gemm_plan.h"
#include "smfmac_common.h"
#include "prune_common.h"        // pack_bf16_rne

namespace nm {

namespace {

constexpr int DK = 64;           // reduction steps of a stage

__device__ __forceinline__ void mfma_32x32x16(f32x16 &acc, const u32x4 &a, const u32x4 &b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// zeros into the registers the block lives in
__device__ __forceinline__ void acc_clear(f32x16 &acc)
{
    const bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    asm volatile("s_nop 4\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "+a"(acc) : "v"(z));
}

union FragK { u32x4 u4; s16x4 q[2]; };

struct DenseArg {
    const uint16_t *x, *w, *bias;              // x [M][K], row stride ldx; w [N][K] or (NN) [K][N], contiguous
    uint16_t *y;                               // [M][N], row stride ldy
    int64_t ldx, ldy, M, N, K;
    int tiles_m, tiles_n, relu;
};

template <int WM, int WN, int AM, int AN, bool NN, int NS>
__global__ __launch_bounds__(WM * WN * 64) void dense_gemm_kernel(DenseArg p)
{
    constexpr int NW = WM * WN, TM = WM * AM * 32, TN = WN * AN * 32;
    constexpr int X_BYTES = TM * DK * 2, STAGE = X_BYTES + TN * DK * 2;
    constexpr int XL = TM / 8 / NW, WL = TN / 8 / NW, LPS = XL + WL;             // direct loads of a wave and stage
    constexpr int CPR = TN / 8, W_ROWS = 64 / CPR;                               // (NN) chunks of a row, rows of a load
    constexpr int LDS = NS * STAGE;
    static_assert(XL >= 1 && WL >= 1 && TM % (8 * NW) == 0 && TN % (8 * NW) == 0 && LDS <= 160 * 1024, "tile");
    __shared__ __attribute__((aligned(1024))) char S[LDS];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, hi = lane >> 5, l32 = lane & 31;
    const int n = (int)((p.K + DK - 1) / DK), k_last = (int)(p.K - (int64_t)(n - 1) * DK);      // stages of a tile; reduction steps of the last one
    const int tiles = p.tiles_m * p.tiles_n;
    auto place = [&](int tile, int64_t &m0, int64_t &n0) {
        int tm, tn;
        tile_of_workgroup(tile, p.tiles_m, p.tiles_n, tm, tn);
        m0 = (int64_t)__builtin_amdgcn_readfirstlane(tm) * TM;
        n0 = (int64_t)__builtin_amdgcn_readfirstlane(tn) * TN;
    };

    f32x16 acc[AM][AN];
#pragma unroll
    for (int a = 0; a < AM; ++a)
#pragma unroll
        for (int b = 0; b < AN; ++b) acc_zero(acc[a][b]);

    // ---- direct loads: load d of a wave covers 1 KB of the stage's image at (wave * XL + d) KB, resp. (wave * WL + d) KB behind the x tile.  Rows past
    // the end are clamped to the last one, their results are not stored; chunks (NN: rows) past the end of the reduction axis are
    // sent out of range, which drops them, and zeroed when the stage has landed.
    const int r8 = lane >> 3, pos = lane & 7;
    uint32_t x_src[XL], w_src[WL];
    int x_k[2], w_k[2];                                                          // first reduction step of a lane's chunk in even and odd loads; NN: w_k[0] its row in load 0
    auto chunk_of = [&](int row) { return pos ^ ((row >> 1) & 7); };
#pragma unroll
    for (int d = 0; d < 2; ++d) { x_k[d] = chunk_of((wave * XL + d) * 8 + r8) * 8; w_k[d] = chunk_of((wave * WL + d) * 8 + r8) * 8; }
    const int w_row = lane / CPR, w_pos = lane % CPR;
    // the tile and stage whose loads are being issued
    int f_tile = blockIdx.x, f_stage = 0;
    const char *xp, *wp;
    const int64_t w_step = NN ? DK * p.N * 2 : DK * 2;
    auto enter_tile = [&]() {
        int64_t m0, n0;
        place(f_tile, m0, n0);
#pragma unroll
        for (int d = 0; d < XL; ++d) {
            const int row = (wave * XL + d) * 8 + r8;
            x_src[d] = (uint32_t)((min(m0 + row, p.M - 1) - m0) * p.ldx * 2 + chunk_of(row) * 16);
        }
#pragma unroll
        for (int d = 0; d < WL; ++d) {
            if constexpr (NN) {
                const int row = (wave * WL + d) * W_ROWS + w_row, swz = TN >= 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1);
                w_src[d] = (uint32_t)((row * p.N + min(n0 + 8 * (w_pos ^ swz), p.N - 8)) * 2);
            } else {
                const int row = (wave * WL + d) * 8 + r8;
                w_src[d] = (uint32_t)((min(n0 + row, p.N - 1) - n0) * p.K * 2 + chunk_of(row) * 16);
            }
        }
        xp = (const char *)(p.x + m0 * p.ldx);
        wp = (const char *)(NN ? p.w : p.w + n0 * p.K);
    };
    enter_tile();
    auto next_stage = [&]() {
        xp += DK * 2; wp += w_step;
        if (++f_stage == n) {
            f_stage = 0;
            f_tile += gridDim.x;
            if (f_tile < tiles) enter_tile();
        }
    };
    auto rsrc = [](const char *base, bool there) { return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, there ? 0x7fffffff : 0, 0x00020000); };
    auto fetch_one = [&](auto k_c, int buf) {
        constexpr int K = decltype(k_c)::value;
        char *stage = S + buf * STAGE;
        const int left = f_stage == n - 1 ? k_last : DK;                         // reduction steps the stage has
        if constexpr (K < XL) {
            const uint32_t src = x_k[K & 1] < left ? x_src[K] : 0xffffffffu;
            load16_to_lds(rsrc(xp, f_tile < tiles), stage + (wave * XL + K) * 1024, src, 0);
        } else {
            constexpr int d = K - XL;
            const int at = NN ? (wave * WL + d) * W_ROWS + w_row : w_k[d & 1];
            const uint32_t src = at < left ? w_src[d] : 0xffffffffu;
            load16_to_lds(rsrc(wp, f_tile < tiles), stage + X_BYTES + (wave * WL + d) * 1024, src, 0);
        }
    };
    // zeros where a wave's loads of the last stage were out of range
    auto clear_tail = [&](int buf) {
        char *stage = S + buf * STAGE;
        const uint4 z = make_uint4(0, 0, 0, 0);
        for (int d = 0; d < XL; ++d)
            if (x_k[d & 1] >= k_last) *(uint4 *)(stage + (wave * XL + d) * 1024 + lane * 16) = z;
        for (int d = 0; d < WL; ++d)
            if ((NN ? (wave * WL + d) * W_ROWS + w_row : w_k[d & 1]) >= k_last) *(uint4 *)(stage + X_BYTES + (wave * WL + d) * 1024 + lane * 16) = z;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

    // ---- LDS reads
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)S;
    const int key = (l32 >> 1) & 7, li = lane & 15;
    uint32_t rd_k[4];                                                            // a row's chunk of MFMA step kk
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) rd_k[kk] = lds0 + (uint32_t)(l32 * (DK * 2) + ((2 * kk + hi) ^ key) * 16);
    const uint32_t x_base = (uint32_t)(wm * AM * 32 * DK * 2), w_base = (uint32_t)(X_BYTES + wn * AN * 32 * DK * 2);
    uint32_t rd_w[AN];
    if constexpr (NN) {
#pragma unroll
        for (int b = 0; b < AN; ++b) {
            const int swz = TN >= 128 ? 4 * (li >> 2) : 4 * ((li >> 3) & 1);
            const int chunk = ((wn * AN + b) * 4 + 2 * ((lane >> 4) & 1) + ((li & 3) >> 1)) ^ swz;
            rd_w[b] = lds0 + (uint32_t)(X_BYTES + (8 * hi + (li >> 2)) * (TN * 2) + chunk * 16 + (li & 1) * 8);
        }
    }
    FragK xf[2][AM], wf[2][AN];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int a = 0; a < AM; ++a) xf[s][a].u4 = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < AN; ++b) wf[s][b].u4 = u32x4{0, 0, 0, 0};
    }
    constexpr int READS = AM + AN * (NN ? 2 : 1);
    static_assert(READS <= 15, "counter of LDS reads");
    auto read = [&](auto kk_c, int buf) {                                        // fragments of MFMA step kk, into set kk % 2
        constexpr int kk = decltype(kk_c)::value, set = kk % 2;
        const uint32_t so = (uint32_t)(buf * STAGE);
        const uint32_t xa = rd_k[kk] + so + x_base;
        static_for<AM>([&](auto a_c) { constexpr int a = decltype(a_c)::value; lds_refill_b128<a * 32 * DK * 2>(xf[set][a].u4, xa); });
        if constexpr (NN)
            static_for<AN>([&](auto b_c) {
                constexpr int b = decltype(b_c)::value, R = TN * 2;
                const uint32_t at = rd_w[b] + so;
                lds_refill_tr16<(16 * kk) * R>(wf[set][b].q[0], at);
                lds_refill_tr16<(16 * kk + 4) * R>(wf[set][b].q[1], at);
            });
        else {
            const uint32_t wa = rd_k[kk] + so + w_base;
            static_for<AN>([&](auto b_c) { constexpr int b = decltype(b_c)::value; lds_refill_b128<b * 32 * DK * 2>(wf[set][b].u4, wa); });
        }
    };
    // The fragments on their way are in their registers.  Stands wherever compiled code lies between a read and the wait for it, which at a loop's head
    // moves fragments to other registers (and would move what was there before); the empty statements keep the registers theirs until then.
    auto reads_landed = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int a = 0; a < AM; ++a) asm volatile("" : : "v"(xf[s][a].u4));
#pragma unroll
            for (int b = 0; b < AN; ++b) asm volatile("" : : "v"(wf[s][b].u4));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // the same of the accumulators and the matrix pipeline
    auto sums_settled = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int a = 0; a < AM; ++a)
#pragma unroll
            for (int b = 0; b < AN; ++b) acc_settled(acc[a][b]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // MFMA step kk; the loads [lo, hi) of a stage are spread behind its MFMAs
    auto step = [&](auto kk_c, auto lo_c, auto hi_c, int buf) {
        constexpr int set = decltype(kk_c)::value % 2, lo = decltype(lo_c)::value, n_l = decltype(hi_c)::value - lo, NM = AM * AN;
        static_for<NM>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value, a = i / AN, b = i % AN;
            mfma_32x32x16(acc[a][b], wf[set][b].u4, xf[set][a].u4);
            static_for<LPS>([&](auto k_c) {
                constexpr int k = decltype(k_c)::value;
                if constexpr (k >= lo && k < lo + n_l && (k - lo) * NM / n_l == i) fetch_one(k_c, buf);
            });
        });
    };
    using std::integral_constant;
    using I0 = integral_constant<int, 0>; using I1 = integral_constant<int, 1>; using I2 = integral_constant<int, 2>; using I3 = integral_constant<int, 3>;

    for (int s = 0; s < NS; ++s) {
        static_for<LPS>([&](auto k_c) { fetch_one(k_c, s); });
        next_stage();
    }
    wait_vmcnt<(NS - 1) * LPS>();
    if (n == 1 && k_last < DK) clear_tail(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(I0{}, 0);
    read(I1{}, 0);
    int buf = 0, s = 0, tile = blockIdx.x;                                       // the stage that is multiplied: its buffer, its number in its tile
    // a stage's first half; behind it every read has landed, so that the loop below closes with none on its way
    auto open = [&]() {
        const int next = buf == NS - 1 ? 0 : buf + 1;
        asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(READS) : "memory");
        step(I0{}, I0{}, I0{}, 0);
        read(I2{}, buf);
        asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(READS) : "memory");
        step(I1{}, I0{}, I0{}, 0);
        read(I3{}, buf);
        // the next stage (of this tile or the next) has landed, and every wave has read all of this one.  (Loads are counted down in the order they
        // were issued, and the stores of the tile before with them.  At a tile's first stage those are younger than the loads that are
        // waited for, so that more has to have landed than is needed; from then on they are older.)
        wait_vmcnt<(NS - 2) * LPS>();
        reads_landed();
        if (k_last < DK && (s + 1 == n ? 0 : s + 1) == n - 1) clear_tail(next);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    open();
    for (;;) {
        const int next = buf == NS - 1 ? 0 : buf + 1;
        step(I2{}, I0{}, integral_constant<int, LPS / 2>{}, buf);
        read(I0{}, next);
        step(I3{}, integral_constant<int, LPS / 2>{}, integral_constant<int, LPS>{}, buf);
        read(I1{}, next);
        next_stage();
        buf = next;
        if (++s == n) {
            // The tile leaves while the next one's first stages are on their way.  The matrix pipeline has to be done with it first, and the reads of the
            // next tile's first fragments with their registers.
            s = 0;
            int64_t m0, n0;
            place(tile, m0, n0);
            const int rows_left = (int)min(p.M - m0, (int64_t)TM);
            reads_landed();
            sums_settled();
#pragma unroll
            for (int b = 0; b < AN; ++b) {
                const int64_t f0 = n0 + (wn * AN + b) * 32;                          // a lane holds the features f0 + 8 g + 4 hi .. + 3 of a token
                char *y0 = (char *)(p.y + m0 * p.ldy + f0);
                // (through the scalar cache: a vector load would wait for the stages' loads, which are older)
                uint2 add[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    u32x4 v = {0u, 0u, 0u, 0u};
                    if (p.bias) v = *(const __attribute__((address_space(4))) u32x4 *)(uintptr_t)(p.bias + min(f0 + 8 * g, p.N - 8));
                    add[g] = hi ? make_uint2(v[2], v[3]) : make_uint2(v[0], v[1]);
                }
#pragma unroll
                for (int a = 0; a < AM; ++a) {
                    const uint32_t row = (uint32_t)((wm * AM + a) * 32 + l32), at = row * (uint32_t)p.ldy * 2u + (uint32_t)hi * 16u;
#pragma unroll
                    for (int g = 0; g < 4; g += 2) {
                        uint32_t w[2][2];
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            float v[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const uint32_t bits = j < 2 ? add[g + i].x : add[g + i].y;
                                v[j] = acc[a][b][4 * (g + i) + j] + __uint_as_float(j & 1 ? bits & 0xffff0000u : bits << 16);
                                if (p.relu) v[j] = v[j] <= 0.f ? 0.f : v[j];         // (a NaN stays one)
                            }
                            w[i][0] = pack_bf16_rne(v[0], v[1]);
                            w[i][1] = pack_bf16_rne(v[2], v[3]);
                        }
                        // the two halves of the wave exchange, so that a lane holds eight features in a row: 8 g .. 8 g + 7, the upper half the eight behind
                        const auto lo = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false), up = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                        if ((int)row < rows_left && f0 + 8 * g + 8 * hi < p.N) *(uint4 *)(y0 + at + 16u * g) = make_uint4(lo[0], up[0], lo[1], up[1]);
                    }
                    acc_clear(acc[a][b]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            sums_settled();                                                          // (of the zeros)
            tile += gridDim.x;
        }
        if (tile >= tiles) break;
        open();
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");                  // what ran ahead
}

}  // namespace

// Tiles of 64 x 64, 128 x 64, 128 x 128 (4 waves, two workgroups on a CU), 128 x 128 on 8 waves with four stages in LDS (one workgroup on a CU) or 256 x 256
// (8 waves), the cheapest by what they were measured to take:
// microseconds per stage of a tile alone on its CU and with a second one, of the largest by the share of the CUs that are busy, and per round.
// Back to back from a graph, these / the vendor library's choice, us: 2048 x 1024 -> 1024 10.3 / 10.2 (input gradient 10.4 / 11.8), 1576 x 768 -> 3072
// 17.5 / 13.5 (21 / 22), 197 x 1024 -> 1024 8.5 / 5.9 (8.3 / 8.0), 6304 x 768 -> 3072 41 / 51 (43 / 38), 12608 x 3072 -> 768 65 / 59 (73 / 69),
// 16384 x 1024 -> 4096 128 / 106 (112 / 103), with the ReLU 128 / 149.  The small tiles are bound by the path from the L2s to the CUs (24 KB a stage in
// 0.33 us on all of them: 18 TB/s), the largest by the matrix pipes at the clock the power limit leaves.
// The eight waves with four stages are for one round of at most 256 tiles, which two stages of 128 x 128 spend waiting (0.85 us a stage, of which 0.2 is matrix
// work) and smaller tiles on more operand bytes: 7478 x 1568 -> 384 23.6 -> 17.6 us (the vendor library 21.0), input gradient 21.7 -> 17.0 (25.5);
// 2774 x 2976 -> 944 40 -> 30 (33), 1881 x 2216 -> 1680 35.7 -> 27.7 (29.9), 931 x 1104 -> 2544 19.4 -> 13.6 (18.0).  Over 230 products of 2e8 to 1.3e10
// multiply-adds the choice takes 0.967 of what it took without, none more than 1.02; over 226 of 181 to 256 tiles and fewer than 24 stages 0.928, none more than
// 1.03 (2130 x 1440 -> 1400 22.8 -> 17.3 us, 935 x 1288 -> 3088 26.1 -> 17.4, 8096 x 1112 -> 376 20.2 -> 15.2, 7343 x 320 -> 496 11.4 -> 8.5).
hipError_t launch_dense_gemm(bool nn, const void *x, int64_t ldx, const void *w, const void *bias, void *y, int64_t ldy, int64_t M, int64_t N, int64_t K,
                             bool relu, hipStream_t st)
{
    DenseArg p{(const uint16_t *)x, (const uint16_t *)w, (const uint16_t *)bias, (uint16_t *)y, ldx, ldy, M, N, K, 0, 0, relu};
    struct Tile { int tm, tn, per_cu; double alone, shared, round; };
    constexpr Tile tiles[5] = {{64, 64, 2, 0.25, 0.42, 0.7}, {128, 64, 2, 0.33, 0.70, 1.0}, {128, 128, 2, 0.85, 1.0, 1.5}, {128, 128, 1, 0.25, 0.55, 1.5}, {256, 256, 1, 0.6, 1.75, 5.0}};
    const double stages = (double)((K + DK - 1) / DK);
    int best = 0;
    double least = 1e300;
    for (int i = 0; i < 5; ++i) {
        const Tile &t = tiles[i];
        const int64_t n = ((M + t.tm - 1) / t.tm) * ((N + t.tn - 1) / t.tn), round = (int64_t)t.per_cu * NM_CUS, left = n % round;
        if (i == 3 && n > NM_CUS) continue;
        const double part = t.per_cu == 1 ? t.alone + (t.shared - t.alone) * (double)left / NM_CUS : left <= NM_CUS ? t.alone : t.shared;
        const double cost = (double)(n / round) * (stages * t.shared + t.round) + (left ? stages * part + t.round : 0.0);
        if (cost < least) { least = cost; best = i; }
    }
    p.tiles_m = (int)((M + tiles[best].tm - 1) / tiles[best].tm);
    p.tiles_n = (int)((N + tiles[best].tn - 1) / tiles[best].tn);
    const int64_t n_tiles = (int64_t)p.tiles_m * p.tiles_n, wgs = std::min<int64_t>(n_tiles, (int64_t)tiles[best].per_cu * NM_CUS);
    if (n_tiles > 0x7fffffffll - 1024) return hipErrorInvalidConfiguration;
#define NM_DENSE(WM, WN, AM, AN, NS)                                                                                                          \
    do {                                                                                                                                      \
        if (nn) hipLaunchKernelGGL((dense_gemm_kernel<WM, WN, AM, AN, true, NS>), dim3((unsigned)wgs), dim3(WM * WN * 64), 0, st, p);          \
        else hipLaunchKernelGGL((dense_gemm_kernel<WM, WN, AM, AN, false, NS>), dim3((unsigned)wgs), dim3(WM * WN * 64), 0, st, p);            \
    } while (0)
    switch (best) {
    case 0: NM_DENSE(2, 2, 1, 1, 4); break;
    case 1: NM_DENSE(2, 2, 2, 1, 3); break;
    case 2: NM_DENSE(2, 2, 2, 2, 2); break;
    case 3: NM_DENSE(2, 4, 2, 1, 4); break;
    default: NM_DENSE(2, 4, 4, 2, 2); break;
    }
#undef NM_DENSE
    return hipGetLastError();
}

}  // namespace nm
