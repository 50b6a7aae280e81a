// Fused MVUE prune + compress kernels for gfx950 (wave64).
//
// One thread owns one 16-token group of VEC columns (VEC = one 16-byte load: 8 bf16 or
// 4 fp32 columns; 4 bf16 columns in the half-width, layer and 8-bit forms).  Blocks (pairs / quads) run along the token axis, i.e. down the rows of
// the thread's own column, so no cross-lane exchange is needed: 16 coalesced 16-byte row
// loads in, 128 contiguous bytes of kept values + VEC 16-bit index words out.
//
// The decision arithmetic is binary32 with one rounding per operation (compiled with
// -ffp-contract=off) so that masks are reproducible bit for bit from (g, seed, stream).
//
//   MVUE 1:2 ........ Sec. 4.1, eq. (6); threshold sampling as in App. B.1
//   optimal 2:4 ..... Sec. 4.2 (eqs. (8), (12), (14)) and App. A.2 (cases 1-3)
//   approx 2:4 ...... Sec. 4.4 (two magnitude-proportional draws, kept value a/p)
//   8-bit output .... Sec. 5 (FP8 neural gradients on top of 2:4), stochastic rounding for the unbiasedness Sec. 3 asks for
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "smfmac_common.h"       // static_for
#include "prune_common.h"
#include "prune_select.h"
#include "q8_scale.h"

namespace nm {

// ------------------------------------------------------------------------------------
// the fused kernel
// ------------------------------------------------------------------------------------
// M = 2: MVUE 1:2; M = 4: EST = 0 the optimal MVUE 2:4, 1 approx-MVUE 2:4, 2 MVUE 1:4; EST = 4 (either M): Greedy;
// DENSE: also write theta(g)
// PROD: the kernel is also the PRODUCER of the neural gradient (eq. (2): g_l = Diag(f'(z_l)) W^T g_{l+1}): g_ holds
// u = W^T g_{l+1} (the dense backward GEMM's output) and dense_ / ldd the derivative factor d = f'(z_l); each row of
// g_l = u * d (one binary32 product per element, rounded to the storage type) is formed in registers, written once to
// gout_ -- the next layer's backward GEMM needs it dense -- and pruned from there: g_l is never read back.
// PROD = 2: the factor is a ReLU's derivative, and d is the layer's OUTPUT y: d = 1 where y > 0, else 0 (nothing writes the factor out).
struct ProdArg { const void *d; int64_t ldd; void *gout; int64_t ldgo; };
// LAYER: the form a layer's backward pass calls (nm_linear_update).  T need not be a multiple of 16: rows past the last token read
// as zeros through the bounds of buffer descriptors (and are not written to gout), so nothing is copied to pad them.  csum (may
// be null): the sum of every column over the thread's 16 rows, csum[G][o], the first half of the bias gradient -- a pass over g
// of its own otherwise.
// Offsets are 32 bits wide, from the first token group of the thread's WAVE: its 64 threads of four columns reach over 32 groups at
// O = 8 and over fewer at any larger O, which at strides up to LAYER_LD_MOST is less than 2^32 bytes.  (From the WORKGROUP's first
// group they would wrap at O = 8 beyond a stride of 2^20, with 32-token groups beyond 2^19.)
struct LayerArg { int64_t T; float *csum; LayerScale scale; };       // scale: the 8-bit form's
static_assert(32 * 32 * LAYER_LD_MOST * 2 <= (int64_t)1 << 32, "32-bit offsets inside a wave: 32 groups of 32 tokens, bf16");
// first token group of the wave's threads
__device__ __forceinline__ int64_t wave_first_group(int64_t ncg)
{
    return ((int64_t)blockIdx.x * 256 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u))) / ncg;
}

// The four column sums of a thread.  No branch on csum: with one, the compiler moves every kept value's arithmetic behind it, and
// all rows stay in registers until there (218 instead of 81); without csum the descriptor is empty and the store is dropped.
// G0: the wave's first token group.
__device__ __forceinline__ void put_csum(const LayerArg &la, int64_t G0, int64_t G, int64_t O, int64_t col0, const float *cs)
{
    const auto r = __builtin_amdgcn_make_buffer_rsrc((char *)(la.csum + G0 * O), 0, la.csum ? 0x7fffffff : 0, 0x00020000);
    const uint4 v = make_uint4(__float_as_uint(cs[0]), __float_as_uint(cs[1]), __float_as_uint(cs[2]), __float_as_uint(cs[3]));
    buffer_put_piece<16>(r, (uint32_t)((G - G0) * O + col0) * 4u, v);
}

template <int DT, int PROD>
__device__ __forceinline__ uint4 producer_row(const uint4 &u, const uint4 &d)
{
    uint4 r;
    auto factor = [](float f) { return PROD == 2 ? (f > 0.0f ? 1.0f : 0.0f) : f; };
    if constexpr (DT == NM_DT_F32) {
        auto mul = [&](uint32_t a, uint32_t b) { return __float_as_uint(__uint_as_float(a) * factor(__uint_as_float(b))); };
        r.x = mul(u.x, d.x); r.y = mul(u.y, d.y); r.z = mul(u.z, d.z); r.w = mul(u.w, d.w);
    } else {
        auto mul2 = [&](uint32_t a, uint32_t b) {
            return pack_bf16_rne(__uint_as_float(a << 16) * factor(__uint_as_float(b << 16)),
                                 __uint_as_float(a & 0xffff0000u) * factor(__uint_as_float(b & 0xffff0000u)));
        };
        r.x = mul2(u.x, d.x); r.y = mul2(u.y, d.y); r.z = mul2(u.z, d.z); r.w = mul2(u.w, d.w);
    }
    return r;
}

// HI0: the caller guarantees that every Philox call index of the launch is below 2^32 (the launcher checks the
// tensor's size): counter words 1-3 are then wave-uniform and the generator's first rounds run partly on the scalar unit.
// CACHED: the streaming form with plain stores, for outputs that the GEMM behind still finds in the L2s
// VEC: columns per thread: one 16-byte load, or half of it (bf16, for launches that would leave SIMDs without work)
template <int DT, int M, int EST, bool DENSE, int PROD = 0, bool HI0 = false, bool NT = false, int VEC = Row<DT>::VEC, bool LAYER = false, bool CACHED = false>
__device__ __forceinline__ void prune_compress_body(
    const void *__restrict__ g_, int64_t n_groups, int64_t O, int64_t ldg,
    uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals_, uint16_t *__restrict__ meta_, void *__restrict__ dense_, int64_t ldd, ProdArg pa = ProdArg{}, LayerArg la = LayerArg{})
{
    static_assert(!(PROD && DENSE), "the producer form writes g_l, not theta(g_l)");
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2;
    constexpr int RB = VEC * ESZ;                     // bytes of a thread's piece of a row: 16 or 8
    const int64_t ncg = O / VEC;
    // (NT: the stores go through whole waves, and the last wave's threads past the end do what the last thread does)
    const int64_t threads = n_groups * ncg, n_own = (int64_t)blockIdx.x * 256 + threadIdx.x, n = NT ? min(n_own, threads - 1) : n_own;
    if ((NT ? n_own - (int64_t)(threadIdx.x & 63) : n) >= threads) return;
    const int64_t G = n / ncg;
    const int64_t col0 = (n - G * ncg) * VEC;

    const char *gp = (const char *)g_ + ((G * 16) * ldg + col0) * ESZ;
    // The second half of the rows is requested only after the first block row is decided (an opaque copy of the
    // address keeps those loads from being hoisted): their latency hides under the arithmetic of the rows already
    // here, and fewer registers are live at once, so one more wave fits each SIMD.
    uint4 rows[16];
    const char *dp_in = nullptr;
    char *gop = nullptr;
    if constexpr (PROD != 0) {
        dp_in = (const char *)pa.d + ((G * 16) * pa.ldd + col0) * ESZ;
        gop = (char *)pa.gout + ((G * 16) * pa.ldgo + col0) * ESZ;
    }
    auto load_piece = [&](const char *p) -> uint4 {
        if constexpr (RB == 16) return NT ? load_stream(p) : load_global(p);
        else return NT ? load_stream8(p) : load_global8(p);
    };
    [[maybe_unused]] float cs[VEC];
    auto add_rows = [&](int r, int n, int c) {            // n rows from r on into the sum of column c
        if constexpr (LAYER) {
            float q = Row<DT>::get(rows[r], c) + Row<DT>::get(rows[r + 1], c);
            if (n == 4) q += Row<DT>::get(rows[r + 2], c) + Row<DT>::get(rows[r + 3], c);
            cs[c] = r == 0 ? q : cs[c] + q;
        }
    };
    auto fetch_rows = [&](const char *base, const char *dbase, int first) {
#pragma unroll
        for (int r = first; r < first + 8; ++r) {
            rows[r] = load_piece(base + (int64_t)r * ldg * ESZ);
            if constexpr (PROD != 0) {
                rows[r] = producer_row<DT, PROD>(rows[r], load_piece(dbase + (int64_t)r * pa.ldd * ESZ));
                if constexpr (NT) store_stream(gop + (int64_t)r * pa.ldgo * ESZ, rows[r]);
                else *(uint4 *)(gop + (int64_t)r * pa.ldgo * ESZ) = rows[r];
            }
        }
    };
    // LAYER: everything through descriptors based at the wave's first token group, with the bytes up to the last token as bound
    // (offsets of 32 bits: see LayerArg)
    [[maybe_unused]] const int64_t t0 = LAYER ? wave_first_group(ncg) * 16 : 0;
    auto rows_rsrc = [&](const void *p, int64_t ld) {
        const int64_t bytes = (la.T - t0) * ld * ESZ;
        return __builtin_amdgcn_make_buffer_rsrc((char *)p + t0 * ld * ESZ, 0, (int)(uint32_t)(bytes > 0xffffffffll ? 0xffffffffll : bytes), 0x00020000);
    };
    auto fetch_rows_layer = [&](uint32_t token, int first) {         // token: G * 16 - t0, through an opaque copy for the second half
        const auto rg = rows_rsrc(g_, ldg);
        const uint32_t og = (token * (uint32_t)ldg + (uint32_t)col0) * ESZ;
#pragma unroll
        for (int r = first; r < first + 8; ++r) rows[r] = buffer_piece<RB>(rg, og + (uint32_t)r * (uint32_t)ldg * ESZ);
        if constexpr (PROD != 0) {
            const auto rd = rows_rsrc(pa.d, pa.ldd), ro = rows_rsrc(pa.gout, pa.ldgo);
            const uint32_t od = (token * (uint32_t)pa.ldd + (uint32_t)col0) * ESZ, oo = (token * (uint32_t)pa.ldgo + (uint32_t)col0) * ESZ;
            uint4 f[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) f[r] = buffer_piece<RB>(rd, od + (uint32_t)(first + r) * (uint32_t)pa.ldd * ESZ);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                rows[first + r] = producer_row<DT, PROD>(rows[first + r], f[r]);
                buffer_put_piece<RB>(ro, oo + (uint32_t)(first + r) * (uint32_t)pa.ldgo * ESZ, rows[first + r]);
            }
        }
    };
    [[maybe_unused]] const uint32_t token0 = (uint32_t)(G * 16 - t0);
    if constexpr (LAYER) fetch_rows_layer(token0, 0);
    else fetch_rows(gp, dp_in, 0);

    // kept values per column in the slot order of the group format, as stored: binary32 words, or bf16 pairs
    // (slots 2i, 2i+1) packed as soon as a block row is decided, which keeps the live registers low
    constexpr int KW = DT == NM_DT_F32 ? 8 : 4;      // words per column
    uint32_t kept[VEC][KW];
    uint32_t md[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) md[c] = 0;
    auto put2 = [&](int c, int i, float v0, float v1) {      // slots 2i and 2i+1 of column c
        if constexpr (DT == NM_DT_F32) { kept[c][2 * i] = __float_as_uint(v0); kept[c][2 * i + 1] = __float_as_uint(v1); }
        else kept[c][i] = pack_bf16_rne(v0, v1);
    };

    constexpr int BLOCK_ROWS = 16 / M;       // pair rows (8) or quad rows (4) in the group
    float held[VEC];                         // 1:2: the kept value of the even pair row, until its partner is known
    // one uniform per block: four blocks share a Philox call (counter blk/4, last counter word 0);
    // approx-MVUE draws twice: two blocks share a call (counter blk/2, last counter word 1)
    constexpr int WPB = EST == 1 ? 2 : 1;            // words per block
    constexpr int CTR_SHIFT = EST == 1 ? 1 : 2;
    constexpr uint32_t DOMAIN = EST == 1 ? 1u : 0u;
    [[maybe_unused]] const uint32_t ctr0 = (uint32_t)(((uint64_t)(G * BLOCK_ROWS) * (uint64_t)O + (uint64_t)col0) >> CTR_SHIFT);   // call index of block row 0
#pragma unroll
    for (int b = 0; b < BLOCK_ROWS; ++b) {
        if (b == 1) {
            if constexpr (LAYER) {
                uint32_t token2 = token0;
                asm volatile("" : "+v"(token2));        // (as below)
                fetch_rows_layer(token2, 8);
            } else {
                const char *gp2 = gp, *dp2 = dp_in;
                asm volatile("" : "+v"(gp2));           // an address the compiler cannot see through
                fetch_rows(gp2, dp2, 8);
            }
        }
        const uint64_t blk0 = (uint64_t)(G * BLOCK_ROWS + b) * (uint64_t)O + (uint64_t)col0;
        uint32_t words[VEC * WPB];
        if constexpr (EST != 4) {
#pragma unroll
            for (int q = 0; q < VEC * WPB / 4; ++q) {
                const uint64_t ctr = (blk0 >> CTR_SHIFT) + q;
                uint32_t w4[4];
                // HI0: the call index fits 32 bits, and block row b adds b * O (a multiple of 8) to the block index
                if constexpr (HI0) philox4x32_10_uniform_c123(ctr0 + (uint32_t)b * (uint32_t)(O >> CTR_SHIFT) + (uint32_t)q, 0u, stream_id, DOMAIN, key0, key1, w4);
                else philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, DOMAIN, key0, key1, w4);
#pragma unroll
                for (int j = 0; j < 4; ++j) words[4 * q + j] = w4[j];
            }
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            if (M == 2) {
                uint32_t k; float v;
                if constexpr (EST == 4) select_greedy_1of2(Row<DT>::get(rows[2 * b], c), Row<DT>::get(rows[2 * b + 1], c), k, v);
                else
                select_1of2(Row<DT>::get(rows[2 * b], c), Row<DT>::get(rows[2 * b + 1], c), words[c], k, v);
                if (b & 1) put2(c, b >> 1, held[c], v); else held[c] = v;
                md[c] |= ((uint32_t)((b & 1) << 1) | k) << (2 * b);
                add_rows(2 * b, 2, c);
            } else {
                float v0, v1; uint32_t nib;
                if constexpr (EST == 1)
                    select_2of4_approx(Row<DT>::get(rows[4 * b], c), Row<DT>::get(rows[4 * b + 1], c),
                                       Row<DT>::get(rows[4 * b + 2], c), Row<DT>::get(rows[4 * b + 3], c),
                                       words[2 * c], words[2 * c + 1], v0, v1, nib);
                else if constexpr (EST == 2)
                    select_1of4(Row<DT>::get(rows[4 * b], c), Row<DT>::get(rows[4 * b + 1], c),
                                Row<DT>::get(rows[4 * b + 2], c), Row<DT>::get(rows[4 * b + 3], c), words[c], v0, v1, nib);
                else if constexpr (EST == 4)
                    select_greedy_2of4<DT>(Key<DT>::make(rows[4 * b], c, 0), Key<DT>::make(rows[4 * b + 1], c, 1),
                                           Key<DT>::make(rows[4 * b + 2], c, 2), Key<DT>::make(rows[4 * b + 3], c, 3), v0, v1, nib);
                else
                    select_2of4<DT>(Key<DT>::make(rows[4 * b], c, 0), Key<DT>::make(rows[4 * b + 1], c, 1),
                                    Key<DT>::make(rows[4 * b + 2], c, 2), Key<DT>::make(rows[4 * b + 3], c, 3),
                                    words[c], v0, v1, nib);
                put2(c, b, v0, v1);
                md[c] |= nib << (4 * b);
                add_rows(4 * b, 4, c);
                __builtin_amdgcn_sched_barrier(0);       // one block at a time: interleaving blocks only lengthens live ranges
            }
        }
    }

    if constexpr (LAYER) {
        static_assert(VEC == 4, "the sums leave as one float4");
        put_csum(la, t0 / 16, G, O, col0, cs);
    }
    // ---- kept values: 8 per column, VEC columns contiguous: 16 PC bytes of a thread (below), of which a wave's 64 threads own one run
    // Streaming stores want whole lines per instruction: the wave's pieces (8 KB at eight columns per thread) go through LDS of
    // its own, written as each thread holds them (PC 16-byte pieces; piece c of lane l at slot PC l + (c ^ l%PC), which spreads the
    // lanes over the banks) and read back so that store k covers bytes [1024 k, 1024 k + 1024).
    // Every lane of the wave is here, and a wave's LDS operations execute in order, so the reads below see the writes above without a
    // workgroup barrier.  The stores go through descriptors that end with the last thread's piece, so that thread counts need be no
    // multiple of 64 (those had plain stores and loads: MVUE 1:2 4112 x 4104 16.9 us, now 12.2, binary32 12208 x 5344 85 -> 64; 2:4 12208 x 1336 17.4 -> 12.9).
    constexpr int PC = VEC * KW / 4;                                     // 16-byte pieces per thread
    uint4 mw;                                                            // index words
    mw.x = md[0] | (md[1] << 16); mw.y = md[2] | (md[3] << 16);
    mw.z = md[4 % VEC] | (md[5 % VEC] << 16); mw.w = md[6 % VEC] | (md[7 % VEC] << 16);
    if constexpr (NT) {
        __shared__ __attribute__((aligned(1024))) char xs[4 * 1024 * PC];
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid) : "v"(kept[VEC - 1][KW - 1]));       // (the addresses below are formed here, after the last block, not carried through the kernel)
        const uint32_t lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6)), wave_lds = wave * (1024 * PC);
        const int64_t n_wave = (int64_t)blockIdx.x * 256 + wave * 64, there = min(threads - n_wave, (int64_t)64);
        // byte address of piece p of this lane: 16 PC lane + 16 (p ^ lane%PC) = (16 PC lane + 16 (lane%PC)) ^ 16 p
        const uint32_t wr = wave_lds + lane * (16 * PC) + (lane % PC) * 16;
#pragma unroll
        for (int c = 0; c < VEC; ++c)
#pragma unroll
            for (int j = 0; j < KW / 4; ++j) {
                const int piece = c * (KW / 4) + j;
                *(uint4 *)(xs + (wr ^ (uint32_t)(piece * 16))) = make_uint4(kept[c][4 * j], kept[c][4 * j + 1], kept[c][4 * j + 2], kept[c][4 * j + 3]);
            }
        __builtin_amdgcn_wave_barrier();
        // store k, lane l: piece l%PC of the wave's thread (64/PC) k + l/PC, which sits at slot 64 k + PC (l/PC) + (l%PC ^ (l/PC)%PC)
        const auto rv = __builtin_amdgcn_make_buffer_rsrc((char *)vals_ + n_wave * (16 * PC), 0, (int)there * (16 * PC), 0x00020000);
        const auto rm = __builtin_amdgcn_make_buffer_rsrc((char *)meta_ + n_wave * (2 * VEC), 0, (int)there * (2 * VEC), 0x00020000);
        const uint32_t rd = wave_lds + (PC * (lane / PC) + ((lane % PC) ^ ((lane / PC) % PC))) * 16;
#pragma unroll
        for (int k = 0; k < PC; ++k) buffer_put_piece<16, !CACHED>(rv, 16 * lane + 1024 * k, *(const uint4 *)(xs + rd + 1024 * k));
        buffer_put_piece<2 * VEC, !CACHED>(rm, 2 * VEC * lane, mw);
    } else {
        uint4 *vp = (uint4 *)((char *)vals_ + n * (16 * PC));
#pragma unroll
        for (int c = 0; c < VEC; ++c)
#pragma unroll
            for (int j = 0; j < KW / 4; ++j) vp[c * (KW / 4) + j] = make_uint4(kept[c][4 * j], kept[c][4 * j + 1], kept[c][4 * j + 2], kept[c][4 * j + 3]);
        if (VEC == 8) *(uint4 *)(meta_ + n * VEC) = mw;
        else *(uint2 *)(meta_ + n * VEC) = make_uint2(mw.x, mw.y);
    }

    // ---- optional dense theta(g)
    if constexpr (DENSE) {
        char *dp = (char *)dense_ + ((G * 16) * ldd + col0) * ESZ;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = r >> 2, p = r & 3;             // quad and position inside it
            uint32_t w[VEC];
#pragma unroll
            for (int c = 0; c < VEC; ++c) {
                const uint32_t nib = (md[c] >> (4 * q)) & 0xfu;
                // the stored words of slots 2q and 2q+1 (bf16: the two halves of one word)
                const uint32_t s0 = DT == NM_DT_F32 ? kept[c][(2 * q) % KW] : (kept[c][q % KW] & 0xffffu);
                const uint32_t s1 = DT == NM_DT_F32 ? kept[c][(2 * q + 1) % KW] : (kept[c][q % KW] >> 16);
                w[c] = (nib & 3u) == (uint32_t)p ? s0 : (nib >> 2) == (uint32_t)p ? s1 : 0u;
            }
            uint4 o;
            if (DT == NM_DT_F32) { o.x = w[0]; o.y = w[1]; o.z = w[2]; o.w = w[3]; }
            else {
                o.x = w[0] | (w[1] << 16); o.y = w[2] | (w[3] << 16);
                o.z = w[4 % VEC] | (w[5 % VEC] << 16); o.w = w[6 % VEC] | (w[7 % VEC] << 16);
            }
            *(uint4 *)(dp + (int64_t)r * ldd * ESZ) = o;
        }
    }
}

// with the dense output
template <int DT, int M, int EST>
__global__ __launch_bounds__(256) void prune_compress_dense_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta, void *__restrict__ dense, int64_t ldd)
{
    prune_compress_body<DT, M, EST, true>(g, n_groups, O, ldg, key0, key1, stream_id, vals, meta, dense, ldd);
}
// Without it, the streaming form: its 32 KB of LDS let five workgroups onto a CU, so five waves per SIMD is
// what the registers are budgeted for (four for the instances that need more than 96).
// HI0: every Philox call index of the launch is below 2^32, which the launcher has checked.
template <int DT, int M, int EST, bool HI0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((DT == NM_DT_BF16 && EST == 1) ? 4 : 5, 5))) void prune_compress_stream_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta)
{
    prune_compress_body<DT, M, EST, false, 0, HI0, true>(g, n_groups, O, ldg, key0, key1, stream_id, vals, meta, nullptr, 0);
}
// Four bf16 columns per thread instead of eight: half the registers and LDS (seven or eight waves per SIMD instead of four or
// five), twice the waves, half the chain of instructions between a wave's loads and its stores.  MVUE 1:2, whose arithmetic is
// light, takes it at every size (32768 x 28672: 495 -> 463 us, 6.3 TB/s; 12608 x 2304: 18.3 -> 16.7; 512 x 512: 5.7 -> 4.0).
// The optimal 2:4 estimator is bound by its arithmetic on large tensors, where the address and index work that two threads do
// instead of one costs 1-2 % (32768 x 28672 530 -> 541 us); below that the launch is a wave or two deep per SIMD and
// what counts is how long one wave takes: 12608 x 768 12.7 -> 9.8, 12608 x 2304 22.3 -> 19.8, 16384 x 4096 41.6 -> 41.0.  Hence the line at 16384 x 4096.
// (Approx-MVUE 2:4 and small tensors: the kernel below.)
constexpr int64_t HALF_MOST = (int64_t)16384 * 4096;        // elements
// Plain stores (CACHED) leave the kept values in the caches for the GEMM behind, streaming ones leave there what else it reads.  Which is the better depends on
// what the program holds there, and not on T and O alone: prune and GEMM in a loop over two sets of tensors, streaming / plain, 2128 x 6496 x 1240 56.7 / 52.6 us,
// 5952 x 2152 x 2304 72 / 65, 8192 x 1536 x 1536 53.3 / 51.0, 9952 x 1760 x 5848 189.7 / 191.9, 16384 x 1024 x 4096 113.8 / 116.2; four layers of a block one after
// the other, 8192 tokens of width 768 202 / 208, 4096 of 1024 171 / 177, 4112 of 1032 182.7 / 194.5, 12208 of 1336 570 / 566.  A launch is left with the
// stores that it had before the streaming form took thread counts that are no multiple of a wave, since either change loses somewhere: whole waves stream,
// and those of a last wave that is not whole store plainly up to 20 Mi elements.  (What the line costs: 4112 of 1032 above, which took 200 with plain
// loads as well.)  A layer's backward pass the same, forward and backward of a layer, streaming / plain: 4531 x 1392 -> 3728 with the ReLU 265 / 254,
// 3682 x 1744 -> 2896 197 / 189, 6058 x 1504 -> 2320 185 / 178, beyond the line 8892 x 496 -> 1976 132 / 133, 14555 x 320 -> 3816 250 / 255.
constexpr int64_t CACHED_MOST = (int64_t)20 << 20;          // elements
template <int M, int EST, bool HI0, bool CACHED = false>
__global__ __launch_bounds__(256) void prune_compress_half_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta)
{
    prune_compress_body<NM_DT_BF16, M, EST, false, 0, HI0, true, 4, false, CACHED>(g, n_groups, O, ldg, key0, key1, stream_id, vals, meta, nullptr, 0);
}
// The value of the lane at distance 1 or 2 among four lanes, and that of the Kth of them
template <int D> __device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, D == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);      // quad_perm [1, 0, 3, 2] or [2, 3, 0, 1]
}
template <int K> __device__ __forceinline__ float lane_of_four(float v)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), K * 0x55, 0xF, 0xF, true));
}

// Four lanes to a token group and four columns, a quad of each column to a lane (the MVUE estimators 2:4 and 1:2, where a lane then has two pairs): four
// times the waves of the kernels above and a quarter of their chain from a wave's loads to its stores, which is what a launch takes that is a few waves
// deep.  The kept pairs are turned among the four lanes, so that a lane stores the eight values of one column.  Call indices below 2^32.
// Graph replays over rotating buffers, the kernel above -> this: optimal 512 x 512 5.3 -> 3.0 us, 1584 x 3072 7.9 -> 6.2, 12608 x 768 10.3 -> 9.7, and past
// the line 8192 x 2048 13.1 -> 13.8, 16384 x 4096 40.7 -> 44.1 (address and index work of four threads instead of one); approx-MVUE,
// whose arithmetic is four times as long, 9.8 -> 4.1, 14.9 -> 9.4, 19.6 -> 15.8, 25 -> 23, 82 -> 79: at every size that the kernel above would take.
// binary32 2:4 1024 x 1024 6.9 -> 3.9, 1376 x 1232 8.2 -> 5.1, 12608 x 768 14.0 -> 12.1, 12608 x 3072 42 -> 37, past the line 16384 x 4096 70.7 -> 74.6
// (approx 10.6 -> 4.8, 11.7 -> 6.3, 20.9 -> 16.9, 58 -> 53, 93.8 -> 96.1); MVUE 1:2, whose chain is shorter, bf16 512 x 512 4.1 -> 2.7, 2288 x 656 7.0 -> 3.5,
// 12608 x 768 9.2 -> 8.6, past the line 4096 x 4096 11.5 -> 11.9, 12608 x 2304 16.7 -> 18.6; binary32 1024 x 1024 4.5 -> 3.2, past it 4096 x 1024 6.0 -> 6.5,
// 8192 x 1024 9.3 -> 10.2 (rows a multiple of 4 KB apart; other widths gain up to 10 % there).
// LAYER, PROD: as in prune_compress_body.
template <int DT, int M, int EST> constexpr int64_t quad_most()          // elements
{
    if (DT == NM_DT_F32) return (int64_t)(M == 2 ? 2 : 40) << 20;
    return EST == 1 ? HALF_MOST : (int64_t)10 << 20;
}
template <int DT, int M, int EST, int PROD = 0, bool LAYER = false>
__global__ __launch_bounds__(256) void prune_compress_quad_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta, ProdArg pa, LayerArg la)
{
    static_assert(PROD == 0 || LAYER, "the producer form of a layer");
    static_assert(!LAYER || DT == NM_DT_BF16, "layers are bf16");
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2, PW = ESZ / 2;           // words of a kept pair
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= n_groups * O) return;                                       // (O is a multiple of 8: the four lanes leave together)
    const int b = (int)(n & 3);                                          // quad
    const uint32_t cell = (uint32_t)(n >> 2), ncg = (uint32_t)(O / 4);
    const uint32_t G = cell / ncg, col0 = (cell - G * ncg) * 4;
    uint4 rows[4];
    // LAYER: the wave's first token group, which the offsets count from (its 16 cells reach over 8 groups at O = 8), as in prune_compress_body
    [[maybe_unused]] const uint32_t G0 = LAYER ? (uint32_t)__builtin_amdgcn_readfirstlane((int)G) : 0u;
    if constexpr (LAYER) {
        const int64_t t0 = (int64_t)G0 * 16;
        auto rows_rsrc = [&](const void *p, int64_t ld) {
            const int64_t bytes = (la.T - t0) * ld * 2;                  // (positive: the wave's first thread has a token)
            return __builtin_amdgcn_make_buffer_rsrc((char *)p + t0 * ld * 2, 0, (int)(uint32_t)(bytes > 0xffffffffll ? 0xffffffffll : bytes), 0x00020000);
        };
        const uint32_t token = (G - G0) * 16 + 4 * b;
        const auto rg = rows_rsrc(g, ldg);
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = buffer_piece<8>(rg, ((token + r) * (uint32_t)ldg + col0) * 2u);
        if constexpr (PROD != 0) {
            const auto rd = rows_rsrc(pa.d, pa.ldd), ro = rows_rsrc(pa.gout, pa.ldgo);
            uint4 f[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) f[r] = buffer_piece<8>(rd, ((token + r) * (uint32_t)pa.ldd + col0) * 2u);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rows[r] = producer_row<NM_DT_BF16, PROD>(rows[r], f[r]);
                buffer_put_piece<8>(ro, ((token + r) * (uint32_t)pa.ldgo + col0) * 2u, rows[r]);
            }
        }
    } else {
        const char *gp = (const char *)g + (((int64_t)G * 16 + 4 * b) * ldg + col0) * ESZ;
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = ESZ == 4 ? load_global(gp + (int64_t)r * ldg * ESZ) : load_global8(gp + (int64_t)r * ldg * ESZ);
    }
    // M = 4: the quad's one call (approx-MVUE: two, side by side); M = 2: one for each of its two rows of pairs
    constexpr int CALLS = EST == 1 || M == 2 ? 2 : 1;
    uint32_t words[4 * CALLS];
#pragma unroll
    for (int q = 0; q < CALLS; ++q) {
        const uint32_t call = M == 2 ? (G * 8 + 2 * b + q) * ncg + col0 / 4 : ((G * 4 + b) * ncg + col0 / 4) * CALLS + q;
        uint32_t w4[4];
        philox4x32_10_uniform_c123(call, 0u, stream_id, EST == 1 ? 1u : 0u, key0, key1, w4);
#pragma unroll
        for (int j = 0; j < 4; ++j) words[4 * q + j] = w4[j];
    }
    uint32_t w[PW][4], nib[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        float v0, v1;
        if constexpr (M == 2) {
            uint32_t k0, k1;
            select_1of2(Row<DT>::get(rows[0], c), Row<DT>::get(rows[1], c), words[c], k0, v0);
            select_1of2(Row<DT>::get(rows[2], c), Row<DT>::get(rows[3], c), words[4 + c], k1, v1);
            nib[c] = k0 | (2u | k1) << 2;
        } else if constexpr (EST == 1)
            select_2of4_approx(Row<DT>::get(rows[0], c), Row<DT>::get(rows[1], c), Row<DT>::get(rows[2], c),
                               Row<DT>::get(rows[3], c), words[2 * c], words[2 * c + 1], v0, v1, nib[c]);
        else
            select_2of4<DT>(Key<DT>::make(rows[0], c, 0), Key<DT>::make(rows[1], c, 1), Key<DT>::make(rows[2], c, 2), Key<DT>::make(rows[3], c, 3),
                            words[c], v0, v1, nib[c]);
        if constexpr (DT == NM_DT_F32) { w[0][c] = __float_as_uint(v0); w[PW - 1][c] = __float_as_uint(v1); }
        else w[0][c] = pack_bf16_rne(v0, v1);
    }
    if constexpr (LAYER) {                                               // column sums: quads (M = 2: pairs) in order, as one thread adds them
        float cs[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float q0 = Row<DT>::get(rows[0], c) + Row<DT>::get(rows[1], c), q1 = Row<DT>::get(rows[2], c) + Row<DT>::get(rows[3], c);
            if constexpr (M == 2) {
                cs[c] = lane_of_four<0>(q0) + lane_of_four<0>(q1);
                cs[c] += lane_of_four<1>(q0); cs[c] += lane_of_four<1>(q1);
                cs[c] += lane_of_four<2>(q0); cs[c] += lane_of_four<2>(q1);
                cs[c] += lane_of_four<3>(q0); cs[c] += lane_of_four<3>(q1);
            } else {
                const float q = q0 + q1;
                cs[c] = lane_of_four<0>(q) + lane_of_four<1>(q);
                cs[c] += lane_of_four<2>(q);
                cs[c] += lane_of_four<3>(q);
            }
        }
        if (b == 0) put_csum(la, G0, G, O, col0, cs);
    }
    // lane b, word c -> lane c, word b
#pragma unroll
    for (int p = 0; p < PW; ++p) {
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            const uint32_t t = lane_xor<1>(b & 1 ? w[p][i] : w[p][i + 1]);
            w[p][i] = b & 1 ? t : w[p][i];
            w[p][i + 1] = b & 1 ? w[p][i + 1] : t;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t t = lane_xor<2>(b & 2 ? w[p][i] : w[p][i + 2]);
            w[p][i] = b & 2 ? t : w[p][i];
            w[p][i + 2] = b & 2 ? w[p][i + 2] : t;
        }
    }
    uint4 *vp = (uint4 *)((char *)vals + n * (8 * ESZ));                 // ((G O + col0 + b) 8 values)
    if constexpr (DT == NM_DT_F32) {
        vp[0] = make_uint4(w[0][0], w[PW - 1][0], w[0][1], w[PW - 1][1]);
        vp[1] = make_uint4(w[0][2], w[PW - 1][2], w[0][3], w[PW - 1][3]);
    } else *vp = make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]);
    uint32_t lo = (nib[0] | (nib[1] << 16)) << (4 * b), hi = (nib[2] | (nib[3] << 16)) << (4 * b);
    lo |= lane_xor<1>(lo); hi |= lane_xor<1>(hi);
    lo |= lane_xor<2>(lo); hi |= lane_xor<2>(hi);
    if (b == 0) *(uint2 *)(meta + n) = make_uint2(lo, hi);
}
// the form of a layer's backward pass (bf16; see LayerArg): PROD = 2 with the ReLU's derivative in front, else 0
template <int M, int EST, int PROD, bool CACHED>
__global__ __launch_bounds__(256) void prune_layer_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta, ProdArg pa, LayerArg la)
{
    prune_compress_body<NM_DT_BF16, M, EST, false, PROD, true, true, 4, true, CACHED>(g, n_groups, O, ldg, key0, key1, stream_id, vals, meta, nullptr, 0, pa, la);
}
// The producer's form.  With plain loads and stores (NT false) where the last wave is not whole, up to 32 Mi elements: with the streaming ones such launches took,
// plain -> streaming, 656 x 1144 11.7 -> 14.5 us, 672 x 1264 11.7 -> 16.7, 3024 x 1144 15.8 -> 18.4, 5408 x 1704 20.5 -> 23.4, 6000 x 5352 49.5 -> 51.4, beyond the line
// 8944 x 8088 124 -> 112 (MVUE 2:4 in bf16; approx-MVUE and binary32 alike, MVUE 1:2 up to 1.3 of the time and, at 14032 x 5216, 0.83).
// Three waves per SIMD are what the streaming form's loads in flight are worth for MVUE 1:2 in bf16 and approx-MVUE in binary32 (153 and 148 registers); left to
// itself the compiler, with the clamped last wave, takes 131 and 96 and more trips to memory: 1536 x 7680 20.9 -> 22.8 us, 512 x 512 13.3 -> 13.9, 12832 x 1408 58.9 -> 63.7.
constexpr int64_t PRODUCER_PLAIN_MOST = (int64_t)32 << 20;  // elements
constexpr bool producer_few_waves(int dt, int m, int est, bool nt) { return nt && (dt == NM_DT_BF16 ? m == 2 : est == 1); }
template <int DT, int M, int EST, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, producer_few_waves(DT, M, EST, NT) ? 3 : 8))) void prune_producer_kernel(
    const void *__restrict__ u, int64_t n_groups, int64_t O, int64_t ldu, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta, ProdArg pa)
{
    prune_compress_body<DT, M, EST, false, 1, false, NT>(u, n_groups, O, ldu, key0, key1, stream_id, vals, meta, nullptr, 0, pa);
}
// The bf16 optimal-2:4 kernel needs 98 registers as the compiler would have it, two more than let a fifth wave onto
// each SIMD; asked for five waves it fits 96 without spilling.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 5))) void prune_compress_bf16_2of4_stream_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals, uint16_t *__restrict__ meta)
{
    prune_compress_body<NM_DT_BF16, 4, 0, false, 0, true, true>(g, n_groups, O, ldg, key0, key1, stream_id, vals, meta, nullptr, 0);
}

// ------------------------------------------------------------------------------------
// 2:4 prune with 8-bit output (Sec. 5, 8-bit rows: FP8 neural gradients; Sec. 3: the quantiser of a neural
// gradient has to be unbiased).  Selection and kept values as above, in binary32; each kept value is multiplied
// by `scale` and rounded stochastically to e5m2 with 16 random bits: with lo <= |x| < hi neighbours on the e5m2
// grid and f = (|x| - lo)/(hi - lo), the result is hi iff r16 + floor(f * 2^16) >= 2^16.
//   |x| >= 57344 (the largest finite e5m2) saturates; a NaN gives an e5m2 NaN.
// Rounding words: one Philox call per four blocks with last counter word 2, word blk%4; its low half rounds the
// first kept value, its high half the second.
// Output: 32-token groups, vals8[(G*O + o)*16 + 2i + s], meta32[G*O + o] (nibble i = quad i).
// ------------------------------------------------------------------------------------
// HI0: every Philox call index of the launch is below 2^32 (checked by the launcher), see prune_compress_body
// VEC, LAYER: as in prune_compress_body (LAYER: T tokens, rows past them zero; csum [groups][O] or null)
template <int DT, int EST, bool HI0, int VEC = Row<DT>::VEC, bool LAYER = false>
__global__ __launch_bounds__(256) void prune_compress_q8_kernel(
    const void *__restrict__ g_, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    float scale, const float *__restrict__ scale_dev, uint8_t *__restrict__ vals8, uint32_t *__restrict__ meta32, LayerArg la)
{
    [[maybe_unused]] uint4 peaks;
    if constexpr (LAYER) peaks = layer_peaks(la.scale);
    else if (scale_dev) scale = scale_dev[0];       // the scale as a device value (element 0 of a scale record)
    auto philox = [&](uint64_t ctr, uint32_t domain, uint32_t (&w4)[4]) {
        if constexpr (HI0) philox4x32_10_uniform_c123((uint32_t)ctr, 0u, stream_id, domain, key0, key1, w4);
        else philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, domain, key0, key1, w4);
    };
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2, RB = VEC * ESZ;
    const int64_t ncg = O / VEC;
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // (LAYER: the last wave's threads past the end stay until it has its scale; what they load is past the last token and reads as zeros)
    if ((LAYER ? n - (int64_t)(threadIdx.x & 63) : n) >= n_groups * ncg) return;
    const int64_t G = n / ncg;
    const int64_t col0 = (n - G * ncg) * VEC;
    const char *gp = (const char *)g_ + ((G * 32) * ldg + col0) * ESZ;

    // rows live in two halves of 8 (two quad rows each); a half is refilled with the rows 16 further down as soon
    // as its quads are decided, through an address the compiler cannot see through (keeps the loads where they are)
    uint4 rows[16];
    [[maybe_unused]] float cs[VEC];
    [[maybe_unused]] const int64_t t0 = LAYER ? wave_first_group(ncg) * 32 : 0;           // (as in prune_compress_body)
    auto fetch_rows = [&](int first) {                                                    // tensor rows first .. first + 7 of the group
        if constexpr (LAYER) {
            const int64_t bytes = (la.T - t0) * ldg * ESZ;
            const auto rg = __builtin_amdgcn_make_buffer_rsrc((char *)g_ + t0 * ldg * ESZ, 0, (int)(uint32_t)(bytes > 0xffffffffll ? 0xffffffffll : bytes), 0x00020000);
            uint32_t token = (uint32_t)(G * 32 - t0);
            if (first) asm volatile("" : "+v"(token));
            const uint32_t og = (token * (uint32_t)ldg + (uint32_t)col0) * ESZ;
#pragma unroll
            for (int r = 0; r < 8; ++r) rows[(first + r) % 16] = buffer_piece<RB>(rg, og + (uint32_t)(first + r) * (uint32_t)ldg * ESZ);
        } else {
            const char *gp2 = gp;
            if (first) asm volatile("" : "+v"(gp2));
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const char *p = gp2 + (int64_t)(first + r) * ldg * ESZ;
                rows[(first + r) % 16] = RB == 16 ? load_global(p) : load_global8(p);
            }
        }
    };
    fetch_rows(0);
    if constexpr (LAYER) {
        scale = layer_scale(la.scale, peaks, blockIdx.x == 0);
        if (n >= n_groups * ncg) return;
    }

    auto add_column = [&](auto b_c, int c) {             // the four rows of quad row b into the column's sum
        if constexpr (LAYER) {
            constexpr int r = (4 * decltype(b_c)::value) % 16;
            const float q = (Row<DT>::get(rows[r], c) + Row<DT>::get(rows[r + 1], c)) + (Row<DT>::get(rows[r + 2], c) + Row<DT>::get(rows[r + 3], c));
            cs[c] = decltype(b_c)::value == 0 ? q : cs[c] + q;
        }
    };
    uint32_t kept[VEC][4];        // 16 e5m2 codes per column
    uint32_t md[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) { md[c] = 0; kept[c][0] = kept[c][1] = kept[c][2] = kept[c][3] = 0; }

    static_for<8>([&](auto b_c) {                       // quad row b: tensor rows 4b .. 4b+3, held in rows[(4b) % 16 ..]
        constexpr int b = decltype(b_c)::value;
        if constexpr (b == 1 || b == 2 || b == 4) fetch_rows(b == 1 ? 8 : b == 2 ? 16 : 24);
        constexpr int R0 = (4 * b) % 16;
        if constexpr (EST == 3) {
            // MVUE 1:2: the quad row holds two pair rows; the kept value of pair row 2b+pr is slot pr of quad b, rounded
            // with the low half of the pair block's rounding word
            static_for<2>([&](auto pr_c) {
                constexpr int pr = decltype(pr_c)::value;
                const uint64_t pblk0 = (uint64_t)(G * 16 + 2 * b + pr) * (uint64_t)O + (uint64_t)col0;
                uint32_t sel[VEC], rnd1[VEC];
#pragma unroll
                for (int q = 0; q < VEC / 4; ++q) {
                    const uint64_t ctr = (pblk0 >> 2) + q;
                    uint32_t w4[4];
                    philox(ctr, 0u, w4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) sel[4 * q + j] = w4[j];
                    philox(ctr, 2u, w4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) rnd1[4 * q + j] = w4[j];
                }
#pragma unroll
                for (int c = 0; c < VEC; ++c) {
                    uint32_t k; float v;
                    select_1of2(Row<DT>::get(rows[R0 + 2 * pr], c), Row<DT>::get(rows[R0 + 2 * pr + 1], c), sel[c], k, v);
                    kept[c][b / 2] = sr_e5m2_into<2 * (b & 1) + pr>(kept[c][b / 2], v * scale, rnd1[c] << 16);
                    md[c] |= ((uint32_t)(pr << 1) | k) << (4 * b + 2 * pr);
                    if constexpr (pr == 1) add_column(b_c, c);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            return;
        }
        const uint64_t blk0 = (uint64_t)(G * 8 + b) * (uint64_t)O + (uint64_t)col0;
        constexpr int WPB = EST == 1 ? 2 : 1;
        uint32_t words[VEC * WPB], rnd[VEC];
#pragma unroll
        for (int q = 0; q < VEC * WPB / 4; ++q) {
            const uint64_t ctr = (blk0 >> (EST == 1 ? 1 : 2)) + q;
            uint32_t w4[4];
            philox(ctr, EST == 1 ? 1u : 0u, w4);
#pragma unroll
            for (int j = 0; j < 4; ++j) words[4 * q + j] = w4[j];
        }
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
            const uint64_t ctr = (blk0 >> 2) + q;
            uint32_t w4[4];
            philox(ctr, 2u, w4);
#pragma unroll
            for (int j = 0; j < 4; ++j) rnd[4 * q + j] = w4[j];
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            float v0, v1; uint32_t nib;
            if constexpr (EST == 1)
                select_2of4_approx(Row<DT>::get(rows[R0], c), Row<DT>::get(rows[R0 + 1], c),
                                   Row<DT>::get(rows[R0 + 2], c), Row<DT>::get(rows[R0 + 3], c),
                                   words[2 * c], words[2 * c + 1], v0, v1, nib);
            else
                select_2of4<DT>(Key<DT>::make(rows[R0], c, 0), Key<DT>::make(rows[R0 + 1], c, 1),
                                Key<DT>::make(rows[R0 + 2], c, 2), Key<DT>::make(rows[R0 + 3], c, 3),
                                words[c], v0, v1, nib);
            kept[c][b / 2] = sr_e5m2_into<2 * (b & 1)>(kept[c][b / 2], v0 * scale, rnd[c] << 16);
            kept[c][b / 2] = sr_e5m2_into<2 * (b & 1) + 1>(kept[c][b / 2], v1 * scale, rnd[c] & 0xffff0000u);
            md[c] |= nib << (4 * b);
            add_column(b_c, c);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
    if constexpr (LAYER) {
        static_assert(VEC == 4, "the sums leave as one float4");
        put_csum(la, t0 / 32, G, O, col0, cs);
    }

    // 16 bytes per column, VEC columns contiguous; one index word per column
    uint4 *vp = (uint4 *)(vals8 + (G * O + col0) * 16);
#pragma unroll
    for (int c = 0; c < VEC; ++c) vp[c] = make_uint4(kept[c][0], kept[c][1], kept[c][2], kept[c][3]);
    uint4 *mp = (uint4 *)(meta32 + (G * O + col0));
#pragma unroll
    for (int c = 0; c < VEC / 4; ++c) mp[c] = make_uint4(md[4 * c], md[4 * c + 1], md[4 * c + 2], md[4 * c + 3]);
}

// The value of the lane at distance 4 among eight lanes: half of the row reversed, then four lanes reversed
__device__ __forceinline__ uint32_t lane_xor4(uint32_t v)
{
    const int t = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);                             // row_half_mirror: 7 - lane
    return (uint32_t)__builtin_amdgcn_mov_dpp(t, 0x1B, 0xF, 0xF, true);                                // quad_perm [3, 2, 1, 0]
}

// Eight lanes to a token group and four columns, a quad of each column to a lane, as in prune_compress_quad_kernel: an eighth of the kernel above's
// chain, which is what a launch takes that is a few waves deep.  Call indices below 2^32.
// Graph replays, the kernel above -> this, us: optimal 512 x 512 9.8 -> 3.2, 2592 x 1928 11.1 -> 6.7, 12608 x 768 16.0 -> 11.3, 4096 x 4096 18.1 -> 15.3,
// 12608 x 3072 33.4 -> 32.4, past the line 16384 x 4096 51.2 -> 54.4; approx-MVUE 19.1 -> 4.3, 20.8 -> 10.4, 30.4 -> 17.6, 32.6 -> 26.5, 62.6 -> 55.0,
// at its line 92.4 -> 90.4; MVUE 1:2 7.9 -> 2.8, 9.4 -> 6.0, 14.5 -> 9.9, 16.2 -> 14.9, past its line 30.7 -> 30.7 and 45.9 -> 53.6.
template <int EST> constexpr int64_t quad_q8_most() { return EST == 1 ? HALF_MOST : (int64_t)(EST == 3 ? 32 : 40) << 20; }      // elements
template <int DT, int EST, bool LAYER = false>
__global__ __launch_bounds__(256) void prune_compress_q8_quad_kernel(
    const void *__restrict__ g, int64_t n_groups, int64_t O, int64_t ldg, uint32_t key0, uint32_t key1, uint32_t stream_id,
    float scale, const float *__restrict__ scale_dev, uint8_t *__restrict__ vals8, uint32_t *__restrict__ meta32, LayerArg la)
{
    static_assert(!LAYER || DT == NM_DT_BF16, "layers are bf16");
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2, RB = 4 * ESZ;
    [[maybe_unused]] uint4 peaks;
    if constexpr (LAYER) peaks = layer_peaks(la.scale);
    else if (scale_dev) scale = scale_dev[0];
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x, threads = n_groups * O * 2;
    // (LAYER: the last wave's threads past the end stay until it has its scale; what they load is past the last token and reads as zeros)
    if ((LAYER ? n - (int64_t)(threadIdx.x & 63) : n) >= threads) return;                              // (O is a multiple of 8: the eight lanes leave together)
    const int b = (int)(n & 7);                                                                        // quad
    const uint32_t cell = (uint32_t)(n >> 3), ncg = (uint32_t)(O / 4);
    const uint32_t G = cell / ncg, col0 = (cell - G * ncg) * 4;
    [[maybe_unused]] const uint32_t G0 = LAYER ? (uint32_t)__builtin_amdgcn_readfirstlane((int)G) : 0u;          // as in prune_compress_quad_kernel: at most 4 groups on
    uint4 rows[4];
    if constexpr (LAYER) {
        const int64_t t0 = (int64_t)G0 * 32, bytes = (la.T - t0) * ldg * ESZ;
        const auto rg = __builtin_amdgcn_make_buffer_rsrc((char *)g + t0 * ldg * ESZ, 0, (int)(uint32_t)(bytes > 0xffffffffll ? 0xffffffffll : bytes), 0x00020000);
        const uint32_t token = (G - G0) * 32 + 4 * b;
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = buffer_piece<RB>(rg, ((token + r) * (uint32_t)ldg + col0) * ESZ);
        scale = layer_scale(la.scale, peaks, blockIdx.x == 0);
        if (n >= threads) return;
    } else {
        const char *gp = (const char *)g + (((int64_t)G * 32 + 4 * b) * ldg + col0) * ESZ;
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = RB == 16 ? load_global(gp + (int64_t)r * ldg * ESZ) : load_global8(gp + (int64_t)r * ldg * ESZ);
    }
    // calls of the selection and of the rounding; MVUE 1:2 has one of either for each of the quad's two rows of pairs
    auto draw = [&](uint32_t call, uint32_t domain, uint32_t *words) {
        uint32_t w4[4];
        philox4x32_10_uniform_c123(call, 0u, stream_id, domain, key0, key1, w4);
#pragma unroll
        for (int j = 0; j < 4; ++j) words[j] = w4[j];
    };
    uint32_t words[8], rnd[8];
    const uint32_t quad_call = (G * 8 + b) * ncg + col0 / 4;
    if constexpr (EST == 3) {
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            const uint32_t call = (G * 16 + 2 * b + pr) * ncg + col0 / 4;
            draw(call, 0u, words + 4 * pr);
            draw(call, 2u, rnd + 4 * pr);
        }
    } else {
        if constexpr (EST == 1) { draw(2 * quad_call, 1u, words); draw(2 * quad_call + 1, 1u, words + 4); }
        else draw(quad_call, 0u, words);
        draw(quad_call, 2u, rnd);
    }
    uint32_t w[4], nib[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        float v0, v1;
        uint32_t r0 = rnd[c] << 16, r1 = rnd[c] & 0xffff0000u;
        if constexpr (EST == 3) {
            uint32_t k0, k1;
            select_1of2(Row<DT>::get(rows[0], c), Row<DT>::get(rows[1], c), words[c], k0, v0);
            select_1of2(Row<DT>::get(rows[2], c), Row<DT>::get(rows[3], c), words[4 + c], k1, v1);
            nib[c] = k0 | (2u | k1) << 2;
            r1 = rnd[4 + c] << 16;
        } else if constexpr (EST == 1)
            select_2of4_approx(Row<DT>::get(rows[0], c), Row<DT>::get(rows[1], c), Row<DT>::get(rows[2], c), Row<DT>::get(rows[3], c),
                               words[2 * c], words[2 * c + 1], v0, v1, nib[c]);
        else
            select_2of4<DT>(Key<DT>::make(rows[0], c, 0), Key<DT>::make(rows[1], c, 1), Key<DT>::make(rows[2], c, 2), Key<DT>::make(rows[3], c, 3),
                            words[c], v0, v1, nib[c]);
        w[c] = sr_e5m2_into<1>(sr_e5m2_into<0>(0u, v0 * scale, r0), v1 * scale, r1);
    }
    if constexpr (LAYER) {                                               // column sums: quads in order, as one thread adds them
        float cs[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float q = (Row<DT>::get(rows[0], c) + Row<DT>::get(rows[1], c)) + (Row<DT>::get(rows[2], c) + Row<DT>::get(rows[3], c));
            const float q4 = __uint_as_float(lane_xor4(__float_as_uint(q)));         // lanes 0-3: the quads of lanes 4-7
            cs[c] = lane_of_four<0>(q) + lane_of_four<1>(q);
            cs[c] += lane_of_four<2>(q); cs[c] += lane_of_four<3>(q);
            cs[c] += lane_of_four<0>(q4); cs[c] += lane_of_four<1>(q4);
            cs[c] += lane_of_four<2>(q4); cs[c] += lane_of_four<3>(q4);
        }
        if (b == 0) put_csum(la, G0, G, O, col0, cs);
    }
    // two lanes make a word of four codes; then lane pair i, word of column c -> lane pair c, word i
#pragma unroll
    for (int c = 0; c < 4; ++c) { const uint32_t t = lane_xor<1>(w[c]); w[c] = b & 1 ? t | w[c] << 16 : w[c] | t << 16; }
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const uint32_t t = lane_xor<2>(b & 2 ? w[i] : w[i + 1]);
        w[i] = b & 2 ? t : w[i];
        w[i + 1] = b & 2 ? w[i + 1] : t;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t t = lane_xor4(b & 4 ? w[i] : w[i + 2]);
        w[i] = b & 4 ? t : w[i];
        w[i + 2] = b & 4 ? w[i + 2] : t;
    }
    // each lane of a pair stores half of the column's 16 bytes: eight bytes a lane
    *(uint2 *)(vals8 + n * 8) = b & 1 ? make_uint2(w[2], w[3]) : make_uint2(w[0], w[1]);              // ((G O + col0) 16 + 8 b)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        nib[c] <<= 4 * b;
        nib[c] |= lane_xor<1>(nib[c]);
        nib[c] |= lane_xor<2>(nib[c]);
        nib[c] |= lane_xor4(nib[c]);
    }
    if (b == 0) *(uint4 *)(meta32 + (n >> 1)) = make_uint4(nib[0], nib[1], nib[2], nib[3]);          // (G O + col0)
}

template <int DT, int EST>
static hipError_t launch_prune_q8_t(const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed, uint32_t stream_id,
                                    float scale, const float *scale_dev, uint8_t *vals8, uint32_t *meta32, hipStream_t st)
{
    const int64_t groups = T / 32;
    // bf16: four columns per thread (half a 16-byte row load), 70-90 registers and five to seven waves per SIMD where eight columns
    // need 128-149 and leave three or four: optimal 2:4 512 x 512 17.4 -> 9.6 us, 12608 x 768 19.2 -> 15.6, 16384 x 4096 51.5 ->
    // 49.2, 32768 x 28672 622 -> 625; MVUE 1:2 587 -> 582 and approx-MVUE 1258 -> 1143 us on the last.
    constexpr int VEC = 4;
    const int64_t threads = groups * (O / VEC);
    if (threads == 0) return hipSuccess;
    if ((threads + 255) / 256 > 0x7fffffffll) return hipErrorInvalidConfiguration;
    if (T * O <= quad_q8_most<EST>()) {
        hipLaunchKernelGGL((prune_compress_q8_quad_kernel<DT, EST>), dim3((unsigned)((groups * O * 2 + 255) / 256)), dim3(256), 0, st,
                           g, groups, O, ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, scale, scale_dev, vals8, meta32, LayerArg{});
        return hipGetLastError();
    }
#define NM_Q8(HI0)                                                                                                                   \
    hipLaunchKernelGGL((prune_compress_q8_kernel<DT, EST, HI0, VEC>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,     \
                       g, groups, O, ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, scale, scale_dev, vals8, meta32, LayerArg{})
    // call indices are at most T*O/8 (approx-MVUE and MVUE 1:2 make more of them than the optimal estimator); the binary32
    // instances run the general code at every size
    if (DT == NM_DT_BF16 && (uint64_t)T * (uint64_t)O <= ((uint64_t)1 << 34)) NM_Q8(DT == NM_DT_BF16);
    else NM_Q8(false);
#undef NM_Q8
    return hipGetLastError();
}

// a layer's 8-bit prune (bf16, T tokens, T not necessarily a multiple of 32; T * O <= 2^34): est 0 optimal 2:4, 1 approx-MVUE 2:4,
// 3 MVUE 1:2; csum (may be null): [ceil(T/32)][O] column sums of g per token group
hipError_t launch_prune_q8_layer(int est, const void *g, int64_t ldg, int64_t T, int64_t O, uint64_t seed, uint32_t stream_id,
                                 const LayerScale &ls, uint8_t *vals8, uint32_t *meta32, float *csum, hipStream_t st)
{
    const int64_t groups = (T + 31) / 32, threads = groups * (O / 4), blocks = (threads + 255) / 256;
    if (threads == 0) return hipSuccess;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
#define NM_Q8L(EST)                                                                                                                     \
    do {                                                                                                                                \
        if (T * O <= quad_q8_most<EST>())                                                                                               \
            hipLaunchKernelGGL((prune_compress_q8_quad_kernel<NM_DT_BF16, EST, true>), dim3((unsigned)((groups * O * 2 + 255) / 256)), dim3(256), 0, st, g, \
                               groups, O, ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, 1.0f, (const float *)nullptr, vals8, meta32, \
                               LayerArg{T, csum, ls});                                                                                  \
        else                                                                                                                            \
            hipLaunchKernelGGL((prune_compress_q8_kernel<NM_DT_BF16, EST, true, 4, true>), dim3((unsigned)blocks), dim3(256), 0, st, g, groups, O, \
                               ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, 1.0f, (const float *)nullptr, vals8, meta32, LayerArg{T, csum, ls}); \
    } while (0)
    if (est == 3) NM_Q8L(3); else if (est == 1) NM_Q8L(1); else NM_Q8L(0);
#undef NM_Q8L
    return hipGetLastError();
}

hipError_t launch_prune_q8(int dt, int est, const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed,
                           uint32_t stream_id, float scale, const float *scale_dev, uint8_t *vals8, uint32_t *meta32, hipStream_t st)
{
#define NM_PRUNE8(DT, EST) launch_prune_q8_t<DT, EST>(g, T, O, ldg, seed, stream_id, scale, scale_dev, vals8, meta32, st)
    // est: 0 optimal MVUE 2:4, 1 approx-MVUE 2:4, 3 MVUE 1:2
    if (dt == NM_DT_F32) return est == 3 ? NM_PRUNE8(NM_DT_F32, 3) : est == 1 ? NM_PRUNE8(NM_DT_F32, 1) : NM_PRUNE8(NM_DT_F32, 0);
    return est == 3 ? NM_PRUNE8(NM_DT_BF16, 3) : est == 1 ? NM_PRUNE8(NM_DT_BF16, 1) : NM_PRUNE8(NM_DT_BF16, 0);
#undef NM_PRUNE8
}

// ------------------------------------------------------------------------------------
// MVUE 2:4 (or 1:2) prune + compress of a gradient stored TRANSPOSED: gT is [O x T], tokens contiguous, so a quad
// (a pair) is four (two) adjacent elements of a row.  Same estimators, same random stream and block index (blk = (t/4)*O + o) as the
// kernels above: the output equals theirs on the transposed tensor, bit for bit.
// Workgroup = 16 columns o x 16 token groups; a thread owns one (o, group): it loads the group's 16 tokens as one
// contiguous piece (16 threads of a column read 512 or 1024 consecutive bytes), decides its four quads, and the
// kept values and index words go through LDS so that the stores run along o (16 x 16 or 32 bytes contiguous per
// token group), which is how the group format is laid out.
// ------------------------------------------------------------------------------------
template <int DT, int EST>
__global__ __launch_bounds__(256) void prune_compress_t_kernel(
    const void *__restrict__ gT_, int64_t n_groups, int64_t O, int64_t ldt, uint32_t key0, uint32_t key1, uint32_t stream_id,
    void *__restrict__ vals_, uint16_t *__restrict__ meta_)
{
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2;
    constexpr int VW = 16 * ESZ / 4;                       // 32-bit words of a group's 16 tokens: 8 (bf16) or 16 (fp32)
    constexpr int KW = 8 * ESZ / 4;                        // words of its 8 kept values: 4 or 8
    __shared__ uint32_t kept_s[16][16][KW + 1];            // [group][column][word] (+1: no bank conflicts on the way in)
    __shared__ uint16_t meta_s[16][16];
    const int tid = threadIdx.x, oi = tid >> 4, gi = tid & 15;
    // consecutive workgroups walk along the tokens of the same 16 columns
    const int64_t gblocks = (n_groups + 15) / 16;
    const int64_t ob = (int64_t)blockIdx.x / gblocks, gb = (int64_t)blockIdx.x % gblocks;
    const int64_t o = ob * 16 + oi, G = gb * 16 + gi;
    const bool live = o < O && G < n_groups;

    uint32_t w[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) w[j] = 0;
    if (live) {
        const uint4 *src = (const uint4 *)((const char *)gT_ + (o * ldt + G * 16) * ESZ);
#pragma unroll
        for (int j = 0; j < VW / 4; ++j) { const uint4 v = src[j]; w[4 * j] = v.x; w[4 * j + 1] = v.y; w[4 * j + 2] = v.z; w[4 * j + 3] = v.w; }
    }
    auto elem_bits = [&](int t) -> uint32_t {             // token t of the group as binary32 bits
        if constexpr (DT == NM_DT_F32) return w[t];
        else return (t & 1) ? (w[t >> 1] & 0xffff0000u) : (w[t >> 1] << 16);
    };
    // Random words.  A wave holds 4 columns (a multiple of 4 onwards) x 16 groups, and the blocks of those 4 columns
    // in one quad row share their Philox calls (one call for the optimal estimator, two for approx-MVUE), as in the
    // token-major kernels.  Lane (a, gi) makes the calls of quad row a of group gi for the wave's columns and leaves
    // the words in LDS; lane (j, gi) then picks, for each quad row, the words of its own column j.
    constexpr int WPC = EST == 1 ? 8 : 4;                  // words per (group, block row) of a wave's four columns
    constexpr int RB = EST == 3 ? 8 : 4;                   // block rows of a group: 8 pair rows (1:2) or 4 quad rows
    __shared__ __attribute__((aligned(16))) uint32_t rnd_s[4][RB][16][WPC];      // [wave][block row][group][word]
    {
        const int wave = tid >> 6, a = oi & 3;
#pragma unroll
        for (int rb = 0; rb < RB / 4; ++rb) {
            const int b = a + 4 * rb;
            const uint64_t blk0 = (uint64_t)(G * RB + b) * (uint64_t)O + (uint64_t)(o - a);
#pragma unroll
            for (int c = 0; c < WPC / 4; ++c) {
                uint32_t r4[4];
                const uint64_t ctr = (blk0 >> (EST == 1 ? 1 : 2)) + c;
                philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, EST == 1 ? 1u : 0u, key0, key1, r4);
                *(uint4 *)&rnd_s[wave][b][gi][4 * c] = make_uint4(r4[0], r4[1], r4[2], r4[3]);
            }
        }
    }
    __syncthreads();
    uint32_t md = 0;
    uint32_t kept[KW];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float v0, v1; uint32_t nib;
        if constexpr (EST == 3) {
            // two pairs fill the two slots of quad i: the first keeps position 0 or 1, the second 2 or 3
            uint32_t k0, k1;
            select_1of2(__uint_as_float(elem_bits(4 * i)), __uint_as_float(elem_bits(4 * i + 1)),
                        rnd_s[tid >> 6][2 * i][gi][oi & 3], k0, v0);
            select_1of2(__uint_as_float(elem_bits(4 * i + 2)), __uint_as_float(elem_bits(4 * i + 3)),
                        rnd_s[tid >> 6][2 * i + 1][gi][oi & 3], k1, v1);
            nib = k0 | ((2u | k1) << 2);
        } else {
        const uint32_t *rw = rnd_s[tid >> 6][i][gi];
        if constexpr (EST == 1) {
            const uint2 wab = *(const uint2 *)&rw[2 * (oi & 3)];
            select_2of4_approx(__uint_as_float(elem_bits(4 * i)), __uint_as_float(elem_bits(4 * i + 1)),
                               __uint_as_float(elem_bits(4 * i + 2)), __uint_as_float(elem_bits(4 * i + 3)), wab.x, wab.y, v0, v1, nib);
        } else {
            const uint32_t word = rw[oi & 3];
            // (the ranking keys are built from one-element "rows": the element sits where column 0 of a row would)
            uint4 e[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t b = elem_bits(4 * i + p);
                e[p] = make_uint4(DT == NM_DT_F32 ? b : (b >> 16), 0u, 0u, 0u);
            }
            select_2of4<DT>(Key<DT>::make(e[0], 0, 0), Key<DT>::make(e[1], 0, 1), Key<DT>::make(e[2], 0, 2), Key<DT>::make(e[3], 0, 3),
                            word, v0, v1, nib);
        }
        }
        if constexpr (DT == NM_DT_F32) { kept[2 * i] = __float_as_uint(v0); kept[2 * i + 1] = __float_as_uint(v1); }
        else kept[i] = pack_bf16_rne(v0, v1);
        md |= nib << (4 * i);
    }
#pragma unroll
    for (int j = 0; j < KW; ++j) kept_s[gi][oi][j] = kept[j];
    meta_s[gi][oi] = (uint16_t)md;
    __syncthreads();
    // second half: thread (group gj, column oj) stores what thread (oj, gj) computed: 16 threads write one token group's run along o
    const int gj = tid >> 4, oj = tid & 15;
    const int64_t o2 = ob * 16 + oj, G2 = gb * 16 + gj;
    if (o2 < O && G2 < n_groups) {
        uint32_t *dst = (uint32_t *)((char *)vals_ + ((G2 * O + o2) * 8) * ESZ);
        // streaming stores (16 threads write whole lines; measured 1.5 % faster than plain ones; streaming LOADS of the
        // 32- or 64-byte pieces a thread reads measured no faster)
        store_stream(dst, make_uint4(kept_s[gj][oj][0], kept_s[gj][oj][1], kept_s[gj][oj][2], kept_s[gj][oj][3]));
        if constexpr (KW == 8) store_stream(dst + 4, make_uint4(kept_s[gj][oj][4], kept_s[gj][oj][5], kept_s[gj][oj][6], kept_s[gj][oj][7]));
        meta_[G2 * O + o2] = meta_s[gj][oj];
    }
}

template <int DT, int EST>
static hipError_t launch_prune_t_t(const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed, uint32_t stream_id,
                                   void *vals, uint16_t *meta, hipStream_t st)
{
    const int64_t groups = T / 16;
    if (groups == 0 || O == 0) return hipSuccess;
    const int64_t blocks = ((groups + 15) / 16) * ((O + 15) / 16);
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((prune_compress_t_kernel<DT, EST>), dim3((unsigned)blocks), dim3(256), 0, st, gT, groups, O, ldt, (uint32_t)seed,
                       (uint32_t)(seed >> 32), stream_id, vals, meta);
    return hipGetLastError();
}

hipError_t launch_prune_transposed(int dt, int est, const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed,
                                   uint32_t stream_id, void *vals, uint16_t *meta, hipStream_t st)
{
    // est: 0 optimal MVUE 2:4, 1 approx-MVUE 2:4, 3 MVUE 1:2
#define NM_T_CASE(DT_, EST_) \
    if (dt == DT_ && est == EST_) return launch_prune_t_t<DT_, EST_>(gT, T, O, ldt, seed, stream_id, vals, meta, st)
    NM_T_CASE(NM_DT_F32, 0); NM_T_CASE(NM_DT_F32, 1); NM_T_CASE(NM_DT_F32, 3);
    NM_T_CASE(NM_DT_BF16, 0); NM_T_CASE(NM_DT_BF16, 1); NM_T_CASE(NM_DT_BF16, 3);
#undef NM_T_CASE
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------
// The 8-bit prune of a gradient stored TRANSPOSED (gT [O x T], tokens contiguous): selection, kept values, scaling and
// stochastic rounding as in prune_compress_q8_kernel, with the same random streams and block indices, so the output
// equals that kernel's on the transposed tensor bit for bit.  Same workgroup shape as prune_compress_t_kernel with
// 32-token groups: a thread owns one (column, group), loads the group's 32 tokens as one contiguous piece (64 or 128
// bytes), decides its eight quads (sixteen pairs), and the 16 codes and the index word go through LDS so that the
// stores run along o.
// ------------------------------------------------------------------------------------
template <int DT, int EST>
__global__ __launch_bounds__(256) void prune_compress_q8_t_kernel(
    const void *__restrict__ gT_, int64_t n_groups, int64_t O, int64_t ldt, uint32_t key0, uint32_t key1, uint32_t stream_id,
    float scale, const float *__restrict__ scale_dev, uint8_t *__restrict__ vals8, uint32_t *__restrict__ meta32)
{
    if (scale_dev) scale = scale_dev[0];
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2;
    constexpr int VW = 32 * ESZ / 4;                       // 32-bit words of a group's 32 tokens: 16 (bf16) or 32 (fp32)
    __shared__ uint32_t kept_s[16][16][5];                 // [group][column][word] (+1: no bank conflicts on the way in)
    __shared__ uint32_t meta_s[16][16];
    const int tid = threadIdx.x, oi = tid >> 4, gi = tid & 15;
    const int64_t gblocks = (n_groups + 15) / 16;          // consecutive workgroups walk along the tokens of the same 16 columns
    const int64_t ob = (int64_t)blockIdx.x / gblocks, gb = (int64_t)blockIdx.x % gblocks;
    const int64_t o = ob * 16 + oi, G = gb * 16 + gi;
    const bool live = o < O && G < n_groups;

    uint32_t w[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) w[j] = 0;
    if (live) {
        const uint4 *src = (const uint4 *)((const char *)gT_ + (o * ldt + G * 32) * ESZ);
#pragma unroll
        for (int j = 0; j < VW / 4; ++j) { const uint4 v = src[j]; w[4 * j] = v.x; w[4 * j + 1] = v.y; w[4 * j + 2] = v.z; w[4 * j + 3] = v.w; }
    }
    auto elem_bits = [&](int t) -> uint32_t {             // token t of the group as binary32 bits
        if constexpr (DT == NM_DT_F32) return w[t];
        else return (t & 1) ? (w[t >> 1] & 0xffff0000u) : (w[t >> 1] << 16);
    };
    // Random words, shared as in prune_compress_t_kernel: a wave holds 4 columns x 16 groups; lane (a, gi) makes the
    // calls of block rows a, a + 4, ... of group gi for the wave's four columns -- the selection words (last counter
    // word 0, or 1 with two calls for approx-MVUE) and the rounding words (last counter word 2) -- and leaves them in LDS.
    constexpr int RB = EST == 3 ? 16 : 8;                  // block rows of a group: 16 pair rows (1:2) or 8 quad rows
    constexpr int SELW = EST == 1 ? 8 : 4;                 // selection words per block row of four columns
    constexpr int WPC = SELW + 4;                          // + their four rounding words
    __shared__ __attribute__((aligned(16))) uint32_t rnd_s[4][RB][16][WPC];      // [wave][block row][group][word]
    {
        const int wave = tid >> 6, a = oi & 3;
#pragma unroll
        for (int rb = 0; rb < RB / 4; ++rb) {
            const int b = a + 4 * rb;
            const uint64_t blk0 = (uint64_t)(G * RB + b) * (uint64_t)O + (uint64_t)(o - a);
            uint32_t r4[4];
#pragma unroll
            for (int c = 0; c < SELW / 4; ++c) {
                const uint64_t ctr = (blk0 >> (EST == 1 ? 1 : 2)) + c;
                philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, EST == 1 ? 1u : 0u, key0, key1, r4);
                *(uint4 *)&rnd_s[wave][b][gi][4 * c] = make_uint4(r4[0], r4[1], r4[2], r4[3]);
            }
            const uint64_t ctr = blk0 >> 2;
            philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, 2u, key0, key1, r4);
            *(uint4 *)&rnd_s[wave][b][gi][SELW] = make_uint4(r4[0], r4[1], r4[2], r4[3]);
        }
    }
    __syncthreads();
    uint32_t md = 0;
    uint32_t kept[4] = {0u, 0u, 0u, 0u};
    const int col = oi & 3;
    static_for<8>([&](auto i_c) {                           // quad i of the group: tokens 4i .. 4i+3, codes 2i and 2i+1
        constexpr int i = decltype(i_c)::value;
        float v0, v1; uint32_t nib, r0, r1;                 // r0, r1: rounding bits of the two kept values, in the top half
        if constexpr (EST == 3) {
            const uint32_t *ra = rnd_s[tid >> 6][2 * i][gi], *rb = rnd_s[tid >> 6][2 * i + 1][gi];
            uint32_t k0, k1;
            select_1of2(__uint_as_float(elem_bits(4 * i)), __uint_as_float(elem_bits(4 * i + 1)), ra[col], k0, v0);
            select_1of2(__uint_as_float(elem_bits(4 * i + 2)), __uint_as_float(elem_bits(4 * i + 3)), rb[col], k1, v1);
            nib = k0 | ((2u | k1) << 2);
            r0 = ra[SELW + col] << 16;                      // each pair block rounds with the low half of its own word
            r1 = rb[SELW + col] << 16;
        } else {
            const uint32_t *rw = rnd_s[tid >> 6][i][gi];
            if constexpr (EST == 1) {
                const uint2 wab = *(const uint2 *)&rw[2 * col];
                select_2of4_approx(__uint_as_float(elem_bits(4 * i)), __uint_as_float(elem_bits(4 * i + 1)),
                                   __uint_as_float(elem_bits(4 * i + 2)), __uint_as_float(elem_bits(4 * i + 3)), wab.x, wab.y, v0, v1, nib);
            } else {
                uint4 e[4];                                 // one-element "rows": the element sits where column 0 of a row would
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const uint32_t b = elem_bits(4 * i + p);
                    e[p] = make_uint4(DT == NM_DT_F32 ? b : (b >> 16), 0u, 0u, 0u);
                }
                select_2of4<DT>(Key<DT>::make(e[0], 0, 0), Key<DT>::make(e[1], 0, 1), Key<DT>::make(e[2], 0, 2), Key<DT>::make(e[3], 0, 3),
                                rw[col], v0, v1, nib);
            }
            const uint32_t r = rw[SELW + col];
            r0 = r << 16;
            r1 = r & 0xffff0000u;
        }
        kept[i / 2] = sr_e5m2_into<2 * (i & 1)>(kept[i / 2], v0 * scale, r0);
        kept[i / 2] = sr_e5m2_into<2 * (i & 1) + 1>(kept[i / 2], v1 * scale, r1);
        md |= nib << (4 * i);
    });
#pragma unroll
    for (int j = 0; j < 4; ++j) kept_s[gi][oi][j] = kept[j];
    meta_s[gi][oi] = md;
    __syncthreads();
    // second half: thread (group gj, column oj) stores what thread (oj, gj) computed: 16 threads write one token group's run along o
    const int gj = tid >> 4, oj = tid & 15;
    const int64_t o2 = ob * 16 + oj, G2 = gb * 16 + gj;
    if (o2 < O && G2 < n_groups) {
        *(uint4 *)(vals8 + (G2 * O + o2) * 16) = make_uint4(kept_s[gj][oj][0], kept_s[gj][oj][1], kept_s[gj][oj][2], kept_s[gj][oj][3]);
        meta32[G2 * O + o2] = meta_s[gj][oj];
    }
}

template <int DT, int EST>
static hipError_t launch_prune_q8_t_t(const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed, uint32_t stream_id, float scale,
                                      const float *scale_dev, uint8_t *vals8, uint32_t *meta32, hipStream_t st)
{
    const int64_t groups = T / 32;
    if (groups == 0 || O == 0) return hipSuccess;
    const int64_t blocks = ((groups + 15) / 16) * ((O + 15) / 16);
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((prune_compress_q8_t_kernel<DT, EST>), dim3((unsigned)blocks), dim3(256), 0, st, gT, groups, O, ldt, (uint32_t)seed,
                       (uint32_t)(seed >> 32), stream_id, scale, scale_dev, vals8, meta32);
    return hipGetLastError();
}

hipError_t launch_prune_q8_transposed(int dt, int est, const void *gT, int64_t T, int64_t O, int64_t ldt, uint64_t seed,
                                      uint32_t stream_id, float scale, const float *scale_dev, uint8_t *vals8, uint32_t *meta32,
                                      hipStream_t st)
{
    // est: 0 optimal MVUE 2:4, 1 approx-MVUE 2:4, 3 MVUE 1:2
#define NM_T8_CASE(DT_, EST_) \
    if (dt == DT_ && est == EST_) return launch_prune_q8_t_t<DT_, EST_>(gT, T, O, ldt, seed, stream_id, scale, scale_dev, vals8, meta32, st)
    NM_T8_CASE(NM_DT_F32, 0); NM_T8_CASE(NM_DT_F32, 1); NM_T8_CASE(NM_DT_F32, 3);
    NM_T8_CASE(NM_DT_BF16, 0); NM_T8_CASE(NM_DT_BF16, 1); NM_T8_CASE(NM_DT_BF16, 3);
#undef NM_T8_CASE
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------
// nm_compress: dense n:m tensor -> group format.  Same thread tiling as above.
// ------------------------------------------------------------------------------------
// The per-wave transpose of prune_compress_body as a function: every lane of the wave hands in the eight 16-byte pieces
// it would have stored at vals + 128 n (n = its thread number in the launch); the wave stores them as eight streaming
// stores of 1 KB of whole lines each.  xs: the workgroup's 32 KB of LDS.  Whole waves only.
__device__ __forceinline__ void store_wave_pieces_stream(void *vals_, char *xs, const uint4 (&piece)[8])
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave_lds = (tid >> 6) * 8192;
    const uint32_t wr = wave_lds + lane * 128 + (lane & 7) * 16;         // piece p at slot 8 lane + (p ^ lane % 8)
#pragma unroll
    for (int p = 0; p < 8; ++p) *(uint4 *)(xs + (wr ^ (uint32_t)(p * 16))) = piece[p];
    __builtin_amdgcn_wave_barrier();
    const int64_t n = (int64_t)blockIdx.x * 256 + tid;
    char *wave_base = (char *)vals_ + (n - lane) * 128;
    const uint32_t rd = wave_lds + (8 * (lane >> 3) + ((lane & 7) ^ (lane >> 3))) * 16;
#pragma unroll
    for (int k = 0; k < 8; ++k) store_stream(wave_base + (1024 * k + 16 * lane), *(const uint4 *)(xs + rd + 1024 * k));
}

template <int DT, int M, bool NT = false>
__global__ __launch_bounds__(256) void compress_kernel(
    const void *__restrict__ d_, int64_t n_groups, int64_t O, int64_t ld,
    void *__restrict__ vals_, uint16_t *__restrict__ meta_, int32_t *__restrict__ bad)
{
    constexpr int VEC = Row<DT>::VEC;
    constexpr int ESZ = DT == NM_DT_F32 ? 4 : 2;
    const int64_t ncg = O / VEC;
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= n_groups * ncg) return;
    const int64_t G = n / ncg;
    const int64_t col0 = (n - G * ncg) * VEC;
    const char *gp = (const char *)d_ + ((G * 16) * ld + col0) * ESZ;
    uint4 rows[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) rows[r] = NT ? load_stream(gp + (int64_t)r * ld * ESZ) : load_global(gp + (int64_t)r * ld * ESZ);

    constexpr int KW = DT == NM_DT_F32 ? 8 : 4;      // stored words per column: binary32 values, or bf16 pairs packed at once
    uint32_t kept[VEC][KW];
    uint32_t md[VEC];
    int nbad = 0;
#pragma unroll
    for (int c = 0; c < VEC; ++c) md[c] = 0;
    // quad row by quad row (the rows of a finished one are dead), one quad at a time
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            float x[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) x[p] = Row<DT>::get(rows[4 * i + p], c);
            uint32_t p0, p1;
            if (M == 4) {
                const uint32_t nz = (x[0] != 0.0f ? 1u : 0u) | (x[1] != 0.0f ? 2u : 0u) |
                                    (x[2] != 0.0f ? 4u : 0u) | (x[3] != 0.0f ? 8u : 0u);
                // straight-line: fewer than two non-zeros are padded with the lowest zero positions (one if one is
                // missing, two if both are)
                uint32_t taken = nz;
                const int cnt = __popc(nz);
                nbad += cnt > 2 ? 1 : 0;
                const uint32_t z1 = ~taken & 0xfu;
                taken |= cnt < 2 ? (z1 & (0u - z1)) : 0u;                  // lowest zero
                const uint32_t z2 = ~taken & 0xfu;
                taken |= cnt < 1 ? (z2 & (0u - z2)) : 0u;
                p0 = (uint32_t)__ffs((int)taken) - 1u;
                taken &= taken - 1u;
                p1 = (uint32_t)__ffs((int)taken) - 1u;
            } else {
                const bool n0 = x[0] != 0.0f, n1 = x[1] != 0.0f, n2 = x[2] != 0.0f, n3 = x[3] != 0.0f;
                nbad += (n0 & n1) + (n2 & n3);
                p0 = (n1 & !n0) ? 1u : 0u;
                p1 = (n3 & !n2) ? 3u : 2u;
            }
            // (two levels of selects on the position's bits: written as a chain of comparisons the compiler made branches of it)
            const uint32_t u0 = __float_as_uint(x[0]), u1 = __float_as_uint(x[1]), u2 = __float_as_uint(x[2]), u3 = __float_as_uint(x[3]);
            const uint32_t k0 = (p0 & 2u) ? ((p0 & 1u) ? u3 : u2) : ((p0 & 1u) ? u1 : u0);
            const uint32_t k1 = (p1 & 2u) ? ((p1 & 1u) ? u3 : u2) : ((p1 & 1u) ? u1 : u0);
            if constexpr (DT == NM_DT_F32) { kept[c][2 * i] = k0; kept[c][2 * i + 1] = k1; }
            else kept[c][i] = (k0 >> 16) | (k1 & 0xffff0000u);        // values are bf16 already: the upper half is exact
            md[c] |= (p0 | (p1 << 2)) << (4 * i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    char *vp = (char *)vals_ + ((G * O + col0) * 8) * ESZ;            // = vals_ + 128 n
    uint4 piece[8];                                                   // the thread's 128 bytes of vals
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
        for (int j = 0; j < KW / 4; ++j)
            piece[c * (KW / 4) + j] = make_uint4(kept[c][4 * j], kept[c][4 * j + 1], kept[c][4 * j + 2], kept[c][4 * j + 3]);
    if constexpr (NT) {
        __shared__ __attribute__((aligned(1024))) char xs[4 * 8192];
        store_wave_pieces_stream(vals_, xs, piece);
    } else {
#pragma unroll
        for (int p = 0; p < 8; ++p) ((uint4 *)vp)[p] = piece[p];
    }
    uint16_t *mp = meta_ + (G * O + col0);
    if (VEC == 8) {
        uint4 o;
        o.x = md[0] | (md[1] << 16); o.y = md[2] | (md[3] << 16);
        o.z = md[4 % VEC] | (md[5 % VEC] << 16); o.w = md[6 % VEC] | (md[7 % VEC] << 16);
        *(uint4 *)mp = o;
    } else {
        uint2 o;
        o.x = md[0] | (md[1] << 16); o.y = md[2] | (md[3] << 16);
        *(uint2 *)mp = o;
    }
    if (bad && nbad) atomicAdd(bad, nbad);
}

// ------------------------------------------------------------------------------------
// launchers (called from the C ABI after validation)
// ------------------------------------------------------------------------------------
template <int DT, int M, int EST>
static hipError_t launch_prune_t(const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed, uint32_t stream_id,
                                 void *vals, uint16_t *meta, void *dense, int64_t ldd, hipStream_t st)
{
    const int64_t groups = T / 16, threads = groups * (O / Row<DT>::VEC);
    if (threads == 0) return hipSuccess;
    const int64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    // hi0: every call index (block / 4, or block / 2 for approx-MVUE's two words per block) lies below 2^32
    const bool hi0 = EST != 4 && (uint64_t)(T / M) * (uint64_t)O <= ((uint64_t)1 << (EST == 1 ? 33 : 34));
    const dim3 grid((unsigned)blocks);
#define NM_ARGS g, groups, O, ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta
    if (dense) {
        hipLaunchKernelGGL((prune_compress_dense_kernel<DT, M, EST>), grid, dim3(256), 0, st, NM_ARGS, dense, ldd);
        return hipGetLastError();
    }
    if constexpr (EST == 0 || EST == 1)
        if (T * O <= quad_most<DT, M, EST>()) {
            hipLaunchKernelGGL((prune_compress_quad_kernel<DT, M, EST>), dim3((unsigned)((groups * O + 255) / 256)), dim3(256), 0, st, NM_ARGS,
                               ProdArg{}, LayerArg{});
            return hipGetLastError();
        }
    if constexpr (DT == NM_DT_BF16 && EST == 0) {
        const dim3 half_grid((unsigned)((2 * threads + 255) / 256));
        if (M == 2 && (2 * threads + 255) / 256 > 0x7fffffffll) return hipErrorInvalidConfiguration;
        if (M == 2 || T * O <= HALF_MOST) {                       // (M = 4: hi0 holds at these sizes)
            if (threads % 32 && T * O <= CACHED_MOST) hipLaunchKernelGGL((prune_compress_half_kernel<M, EST, true, true>), half_grid, dim3(256), 0, st, NM_ARGS);
            else if (hi0) hipLaunchKernelGGL((prune_compress_half_kernel<M, EST, true>), half_grid, dim3(256), 0, st, NM_ARGS);
            else if constexpr (M == 2) hipLaunchKernelGGL((prune_compress_half_kernel<M, EST, false>), half_grid, dim3(256), 0, st, NM_ARGS);
        } else if constexpr (M == 4) {
            if (hi0) hipLaunchKernelGGL(prune_compress_bf16_2of4_stream_kernel, grid, dim3(256), 0, st, NM_ARGS);
            else hipLaunchKernelGGL((prune_compress_stream_kernel<DT, M, EST, false>), grid, dim3(256), 0, st, NM_ARGS);
        }
    } else {
        if (hi0) hipLaunchKernelGGL((prune_compress_stream_kernel<DT, M, EST, true>), grid, dim3(256), 0, st, NM_ARGS);
        else hipLaunchKernelGGL((prune_compress_stream_kernel<DT, M, EST, false>), grid, dim3(256), 0, st, NM_ARGS);
    }
#undef NM_ARGS
    return hipGetLastError();
}

// g_l = u * d written to gout, and its prune + compress, in one pass.  m = 2: MVUE 1:2; m = 4: est 0 optimal / 1 approx-MVUE 2:4
hipError_t launch_prune_producer(int dt, int m, int est, const void *u, int64_t ldu, const void *d, int64_t ldd, int64_t T, int64_t O,
                                 uint64_t seed, uint32_t stream_id, void *gout, int64_t ldgo, void *vals, uint16_t *meta, hipStream_t st)
{
    const int64_t groups = T / 16, threads = groups * (O / (dt == NM_DT_F32 ? 4 : 8));
    if (threads == 0) return hipSuccess;
    const int64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    const ProdArg pa{d, ldd, gout, ldgo};
    const bool plain = threads % 64 && T * O <= PRODUCER_PLAIN_MOST;
#define NM_PROD(DT, M, EST)                                                                                                             \
    do {                                                                                                                                \
        if (plain)                                                                                                                      \
            hipLaunchKernelGGL((prune_producer_kernel<DT, M, EST, false>), dim3((unsigned)blocks), dim3(256), 0, st, u, groups, O, ldu, \
                               (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta, pa);                                      \
        else                                                                                                                            \
            hipLaunchKernelGGL((prune_producer_kernel<DT, M, EST, true>), dim3((unsigned)blocks), dim3(256), 0, st, u, groups, O, ldu,  \
                               (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta, pa);                                      \
    } while (0)
    if (dt == NM_DT_F32) { if (m == 2) NM_PROD(NM_DT_F32, 2, 0); else if (est == 1) NM_PROD(NM_DT_F32, 4, 1); else NM_PROD(NM_DT_F32, 4, 0); }
    else { if (m == 2) NM_PROD(NM_DT_BF16, 2, 0); else if (est == 1) NM_PROD(NM_DT_BF16, 4, 1); else NM_PROD(NM_DT_BF16, 4, 0); }
#undef NM_PROD
    return hipGetLastError();
}

// A layer's prune (bf16, T tokens, T not necessarily a multiple of 16; T * O <= 2^34): m = 2: MVUE 1:2; m = 4: est 0 optimal / 1
// approx-MVUE 2:4.  act (may be null): the ReLU's output; g = u * [act > 0] is then written to gout.  csum (may be null):
// [ceil(T/16)][O] column sums of g per token group.
hipError_t launch_prune_layer(int m, int est, const void *g, int64_t ldg, const void *act, int64_t lda, int64_t T, int64_t O, uint64_t seed,
                              uint32_t stream_id, void *gout, int64_t ldgo, void *vals, uint16_t *meta, float *csum, hipStream_t st)
{
    const int64_t groups = (T + 15) / 16, threads = groups * (O / 4), blocks = (threads + 255) / 256;
    if (threads == 0) return hipSuccess;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    const ProdArg pa{act, lda, gout, ldgo};
    const LayerArg la{T, csum};
    const bool cached = threads % 64 && T * O <= CACHED_MOST;
#define NM_LAYER(M, EST, PROD)                                                                                                  \
    do {                                                                                                                        \
        if (cached)                                                                                                             \
            hipLaunchKernelGGL((prune_layer_kernel<M, EST, PROD, true>), dim3((unsigned)blocks), dim3(256), 0, st, g, groups, O, ldg,  \
                               (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta, pa, la);                          \
        else                                                                                                                    \
            hipLaunchKernelGGL((prune_layer_kernel<M, EST, PROD, false>), dim3((unsigned)blocks), dim3(256), 0, st, g, groups, O, ldg, \
                               (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta, pa, la);                          \
    } while (0)
#define NM_QUAD(M, EST, PROD)                                                                                                           \
    hipLaunchKernelGGL((prune_compress_quad_kernel<NM_DT_BF16, M, EST, PROD, true>), dim3((unsigned)((groups * O + 255) / 256)), dim3(256), 0, st, g, groups, O, \
                       ldg, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, vals, meta, pa, la)
    if (m == 4 && est == 1 && T * O <= quad_most<NM_DT_BF16, 4, 1>()) { if (act) NM_QUAD(4, 1, 2); else NM_QUAD(4, 1, 0); }
    else if (m == 4 && est == 0 && T * O <= quad_most<NM_DT_BF16, 4, 0>()) { if (act) NM_QUAD(4, 0, 2); else NM_QUAD(4, 0, 0); }
    else if (m == 2 && T * O <= quad_most<NM_DT_BF16, 2, 0>()) { if (act) NM_QUAD(2, 0, 2); else NM_QUAD(2, 0, 0); }
    else if (act) { if (m == 2) NM_LAYER(2, 0, 2); else if (est == 1) NM_LAYER(4, 1, 2); else NM_LAYER(4, 0, 2); }
    else { if (m == 2) NM_LAYER(2, 0, 0); else if (est == 1) NM_LAYER(4, 1, 0); else NM_LAYER(4, 0, 0); }
#undef NM_QUAD
#undef NM_LAYER
    return hipGetLastError();
}

// m = 2: est = 0 MVUE 1:2, 4 Greedy 1:2;  m = 4: est = 0 optimal MVUE 2:4, 1 approx-MVUE 2:4, 2 MVUE 1:4, 4 Greedy 2:4
hipError_t launch_prune(int dt, int m, int est, const void *g, int64_t T, int64_t O, int64_t ldg, uint64_t seed,
                        uint32_t stream_id, void *vals, uint16_t *meta, void *dense, int64_t ldd, hipStream_t st)
{
#define NM_PRUNE(DT, M, EST) launch_prune_t<DT, M, EST>(g, T, O, ldg, seed, stream_id, vals, meta, dense, ldd, st)
    if (dt == NM_DT_F32) {
        if (m == 2) return est == 4 ? NM_PRUNE(NM_DT_F32, 2, 4) : NM_PRUNE(NM_DT_F32, 2, 0);
        return est == 1 ? NM_PRUNE(NM_DT_F32, 4, 1) : est == 2 ? NM_PRUNE(NM_DT_F32, 4, 2) : est == 4 ? NM_PRUNE(NM_DT_F32, 4, 4) : NM_PRUNE(NM_DT_F32, 4, 0);
    }
    if (m == 2) return est == 4 ? NM_PRUNE(NM_DT_BF16, 2, 4) : NM_PRUNE(NM_DT_BF16, 2, 0);
    return est == 1 ? NM_PRUNE(NM_DT_BF16, 4, 1) : est == 2 ? NM_PRUNE(NM_DT_BF16, 4, 2) : est == 4 ? NM_PRUNE(NM_DT_BF16, 4, 4) : NM_PRUNE(NM_DT_BF16, 4, 0);
#undef NM_PRUNE
}

template <int DT, int M>
static hipError_t launch_compress_t(const void *d, int64_t T, int64_t O, int64_t ld, void *vals, uint16_t *meta,
                                    int32_t *bad, hipStream_t st)
{
    const int64_t groups = T / 16, threads = groups * (O / Row<DT>::VEC);
    if (threads == 0) return hipSuccess;
    if ((threads + 255) / 256 > 0x7fffffffll) return hipErrorInvalidConfiguration;
    if (threads % 64 == 0)          // whole waves: streaming loads, stores of whole lines through the per-wave transpose
        hipLaunchKernelGGL((compress_kernel<DT, M, true>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                           d, groups, O, ld, vals, meta, bad);
    else
        hipLaunchKernelGGL((compress_kernel<DT, M, false>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                           d, groups, O, ld, vals, meta, bad);
    return hipGetLastError();
}

hipError_t launch_compress(int dt, int m, const void *d, int64_t T, int64_t O, int64_t ld, void *vals,
                           uint16_t *meta, int32_t *bad, hipStream_t st)
{
    if (dt == NM_DT_F32)
        return m == 2 ? launch_compress_t<NM_DT_F32, 2>(d, T, O, ld, vals, meta, bad, st)
                      : launch_compress_t<NM_DT_F32, 4>(d, T, O, ld, vals, meta, bad, st);
    return m == 2 ? launch_compress_t<NM_DT_BF16, 2>(d, T, O, ld, vals, meta, bad, st)
                  : launch_compress_t<NM_DT_BF16, 4>(d, T, O, ld, vals, meta, bad, st);
}

}  // namespace nm
