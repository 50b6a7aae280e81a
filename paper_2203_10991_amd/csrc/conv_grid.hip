// The padded channels-last grid of a convolution's update GEMM, straight from the tensors a layer holds.
//
// The update GEMM on shifted views (nm_update_gemm_shifted) wants activations and gradient on one zero-padded grid
// [N][H+2p][W+2p][C] flattened to rows.  One launch makes what it consumes, one pass over each tensor; its workgroups are
// dealt to two tasks:
//   grid_pack    activations [N, C, H, W] (channel planes, or channels last) -> the grid's rows with the zero
//                       border and the zero margin rows, as bf16 or scaled and rounded to e4m3
//   prune_grid   the same grid of the gradient, never written: a tile of it is put together in LDS, pruned 2:4 along the
//                       grid's rows and compressed (16-token groups, bf16) or also rounded to e5m2 (32-token groups)
// Masks and values are those of the ordinary prune on the materialised grid (same block index, same random words).
//
// Bound: HBM (one read of each tensor, one write of each result); alone, the pack is bound by it and the prune by its vector
// arithmetic, so the two tasks alternate workgroup by workgroup (256 x 64 x 56 x 56: 90 us in two launches, 87 in one, the layer
// 142 -> 140 with both sides timed in turn; 8-bit 14 x 14 stage 36.4 -> 33.2, the layer 87.2 -> 84.3).  Streaming loads or stores
// make the layer 4-11 % slower: the memory-side cache serves the next kernel.  Before, the layer made the grid with tensor operations: a fill and a strided permuting copy per padding, a fill and a copy per margin --
// 375 us for the two tensors of a 256 x 64 x 56 x 56 layer, whose bytes take 60 us, then the prune read the grid again.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "nm_internal.h"
#include "smfmac_common.h"       // static_for
#include "prune_common.h"
#include "prune_select.h"
#include "q8_scale.h"

namespace nm {

// Geometry of the grid: row r = (n * Hp + y) * Wp + x; rows outside the image's interior are zero.
struct GridGeom {
    int H, W, C, pad;
    int Hp, Wp;
    int64_t rows;                // N * Hp * Wp
};
inline GridGeom grid_geom(const ConvShape &s, int C)
{
    GridGeom g;
    g.H = s.H; g.W = s.W; g.C = C; g.pad = s.k / 2; g.Hp = s.H + 2 * g.pad; g.Wp = s.W + 2 * g.pad;
    g.rows = (int64_t)s.N * g.Hp * g.Wp;
    return g;
}

// element offset of channel 0 of grid row r in the tensor, or -1 where the grid holds zeros
__device__ __forceinline__ int64_t grid_source(const GridGeom &gg, bool cl, int64_t r)
{
    if (r < 0 || r >= gg.rows) return -1;
    const uint32_t q = (uint32_t)r / (uint32_t)gg.Wp, x = (uint32_t)r - q * (uint32_t)gg.Wp;      // (rows < 2^31: checked by the caller)
    const uint32_t n = q / (uint32_t)gg.Hp, y = q - n * (uint32_t)gg.Hp;
    const int xi = (int)x - gg.pad, yi = (int)y - gg.pad;
    if (xi < 0 || xi >= gg.W || yi < 0 || yi >= gg.H) return -1;
    const int64_t plane = (int64_t)gg.H * gg.W, s = (int64_t)yi * gg.W + xi;
    return cl ? ((int64_t)n * plane + s) * gg.C : (int64_t)n * plane * gg.C + s;
}

// A tile of the grid in LDS: TILE_ROWS rows x TILE_COLS channels, 34 words per row (64 channels and two words of padding: a
// row starts on an 8-byte boundary, and both the row-wise reads and the column-wise writes spread over the banks).
constexpr int TILE_ROWS = 256, TILE_COLS = 64, TILE_LD = TILE_COLS / 2 + 2;

// Channel planes: thread t owns the grid rows r0 + 2p, r0 + 2p+1 (p = t % 128) of half of the channels, so the 64 lanes of a wave read
// runs of consecutive x of one channel, two pixels to a lane in one 4-byte load, at any alignment of 2 bytes; a byte permutation per word
// then puts pairs of channels together (and zeros where a row is border).  Both rows of a thread lie in one image row, or one of
// them is border, where there is a border; without one where a plane has an even number of pixels.  Otherwise (and with images one pixel
// wide) thread t owns row r0 + t.  Half the load instructions of one pixel to a lane: the launch of a 256 x 256 x 14 x 14 8-bit layer 33 -> 28 us,
// of a 256 x 64 x 56 x 56 layer 89 -> 85.  Channels last: eight threads share a row, 16 bytes each.
typedef uint32_t u32_any2 __attribute__((aligned(2), may_alias));      // a 4-byte load from a 2-byte boundary

__device__ __forceinline__ void load_tile(uint32_t *tile, int64_t *offs, const uint16_t *__restrict__ src, const GridGeom &gg, bool cl,
                                          int64_t r0, int c0)
{
    const int tid = threadIdx.x;
    const int cols = min(TILE_COLS, gg.C - c0);                      // a multiple of 8
    const int64_t plane = (int64_t)gg.H * gg.W;
    const bool pairs = gg.pad > 0 ? gg.W >= 2 : plane % 2 == 0;
    if (!cl && pairs) {
        const int pr = tid & 127, n_c = cols / 2, c1 = (tid >> 7) * n_c;      // channels c1 .. c1 + n_c - 1, a multiple of 4
        const int64_t a = grid_source(gg, false, r0 + 2 * pr), b = grid_source(gg, false, r0 + 2 * pr + 1);
        // the loaded pixels are x, x+1 (both rows), x-1, x (the first row only: x ends an image row) or x, x+1 (the second only: x starts one)
        const uint32_t lo = 0x05040100u, hi = 0x07060302u, none = 0x0c0c0c0cu;      // of two words: the low halves, the high halves, zeros
        const uint32_t sel_a = a < 0 ? none : b < 0 ? hi : lo, sel_b = b < 0 ? none : a < 0 ? lo : hi;
        const uint16_t *p = src + (b < 0 ? (a < 0 ? 0 : a - 1) : a < 0 ? b : a) + (int64_t)(c0 + c1) * plane;
        uint32_t *w = tile + 2 * pr * TILE_LD + c1 / 2;
        auto channels = [&](int c, auto n_c_) {                       // n channels from c on, all loads in flight together
            constexpr int n = decltype(n_c_)::value;
            uint32_t v[n];
#pragma unroll
            for (int j = 0; j < n; ++j) v[j] = *(const u32_any2 *)(p + (int64_t)(c + j) * plane);
#pragma unroll
            for (int j = 0; j < n; j += 4) {
                *(uint2 *)(w + (c + j) / 2) = make_uint2(__builtin_amdgcn_perm(v[j + 1], v[j], sel_a), __builtin_amdgcn_perm(v[j + 3], v[j + 2], sel_a));
                *(uint2 *)(w + TILE_LD + (c + j) / 2) = make_uint2(__builtin_amdgcn_perm(v[j + 1], v[j], sel_b), __builtin_amdgcn_perm(v[j + 3], v[j + 2], sel_b));
            }
        };
        int c = 0;
        for (; c + 32 <= n_c; c += 32) channels(c, std::integral_constant<int, 32>{});
        for (; c < n_c; c += 4) channels(c, std::integral_constant<int, 4>{});
        __syncthreads();
        return;
    }
    const int64_t o = grid_source(gg, cl, r0 + tid);
    if (!cl) {
        const uint16_t *p = src + (o < 0 ? 0 : o) + (int64_t)c0 * plane;      // (a border row reads image 0 and drops it)
        const uint32_t keep = o < 0 ? 0u : 0xffffffffu;
        uint32_t *w = tile + tid * TILE_LD;
        auto channels = [&](int c, auto n_c_) {                       // n channels from c on, all loads in flight together (8 at a time: 57 x 256 x 27 x 29 17.4 -> 19.4 us)
            constexpr int n = decltype(n_c_)::value;
            uint32_t v[n];
#pragma unroll
            for (int j = 0; j < n; ++j) v[j] = (uint32_t)p[(int64_t)(c + j) * plane];
#pragma unroll
            for (int j = 0; j < n / 2; ++j) w[c / 2 + j] = (v[2 * j] | (v[2 * j + 1] << 16)) & keep;
        };
        int c = 0;
        for (; c + 32 <= cols; c += 32) channels(c, std::integral_constant<int, 32>{});
        for (; c < cols; c += 8) channels(c, std::integral_constant<int, 8>{});
    } else {
        offs[tid] = o;
        __syncthreads();
        const int piece = tid & 7;
        if (8 * piece < cols) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int row = 32 * k + (tid >> 3);
                const int64_t so = offs[row];
                uint4 v = make_uint4(0, 0, 0, 0);
                if (so >= 0) v = load_global(src + so + c0 + 8 * piece);
                uint2 *w = (uint2 *)(tile + row * TILE_LD + 4 * piece);
                w[0] = make_uint2(v.x, v.y);
                w[1] = make_uint2(v.z, v.w);
            }
        }
    }
    __syncthreads();
}

// ------------------------------------------------------------------------------------
// activations -> rows [-margin, T + margin) of the grid, out row 0 = grid row -margin
// ------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t e4m3_of_words(uint32_t a, uint32_t b, float s)       // two words of two bf16 -> four codes
{
    auto cl = [](float v) { return __builtin_amdgcn_fmed3f(v, -448.0f, 448.0f); };
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(__uint_as_float(a << 16) * s), cl(__uint_as_float(a & 0xffff0000u) * s), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(__uint_as_float(b << 16) * s), cl(__uint_as_float(b & 0xffff0000u) * s), w, true);
    return (uint32_t)w;
}

template <bool Q8>
__device__ __forceinline__ void grid_pack(uint32_t *tile, int64_t *offs, const uint16_t *__restrict__ x, const GridGeom &gg, bool cl, int64_t margin,
                                          int64_t out_rows, const LayerScale &ls, void *__restrict__ out_, int64_t bx, int by)
{
    const int64_t r0 = bx * TILE_ROWS;                                  // out row
    const int c0 = by * TILE_COLS;
    [[maybe_unused]] uint4 peaks;
    if constexpr (Q8) peaks = layer_peaks(ls);
    load_tile(tile, offs, x, gg, cl, r0 - margin, c0);
    float s = 1.0f;
    if constexpr (Q8) s = layer_scale(ls, peaks, bx == 0 && by == 0);
    constexpr int PER = Q8 ? 16 : 8;                                    // channels of a 16-byte piece
    constexpr int PR = TILE_COLS / PER;                                 // pieces per row
#pragma unroll
    for (int k = 0; k < TILE_ROWS * PR / 256; ++k) {
        const int p = k * 256 + threadIdx.x, row = p / PR, piece = p % PR;
        const int c = c0 + piece * PER;
        if (r0 + row >= out_rows || c >= gg.C) continue;
        const uint2 *w = (const uint2 *)(tile + row * TILE_LD + piece * (PER / 2));
        uint4 o;
        if constexpr (Q8) {
            const uint2 a = w[0], b = w[1], d = w[2], e = w[3];
            o = make_uint4(e4m3_of_words(a.x, a.y, s), e4m3_of_words(b.x, b.y, s), e4m3_of_words(d.x, d.y, s), e4m3_of_words(e.x, e.y, s));
            *(uint4 *)((uint8_t *)out_ + (r0 + row) * gg.C + c) = o;
        } else {
            const uint2 a = w[0], b = w[1];
            o = make_uint4(a.x, a.y, b.x, b.y);
            *(uint4 *)((uint16_t *)out_ + (r0 + row) * gg.C + c) = o;
        }
    }
}

// ------------------------------------------------------------------------------------
// gradient -> 2:4 prune + compress along the grid's rows.  EST: 0 optimal MVUE, 1 approx-MVUE.
// A workgroup takes 256 grid rows x 64 channels through its LDS tile.  bf16: a thread owns one 16-token group of four columns, the
// columns that share Philox calls.  8-bit (Q8): a 32-token group of TWO columns -- four would leave half the threads of a tile without
// work -- and two neighbouring lanes share the calls of their four columns: the even lane makes the selection call, the odd
// lane the rounding call, and they exchange the halves.
// Kept values leave through the wave's own part of the tile (its rows are read by no other wave), so that every store
// instruction covers whole lines: 64 columns of one group, 1 KB.
// HI0: every Philox call index of the launch is below 2^32.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t swap_pair(uint32_t v)              // the value of the neighbouring lane (lane ^ 1)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);      // quad_perm [1, 0, 3, 2]
}

template <int EST>
__device__ __forceinline__ void select_quad_bf16(const uint32_t (&w)[4], int half, uint32_t word1, uint32_t word2, float &v0, float &v1, uint32_t &nib)
{
    // w: the four tokens' words; `half` picks the column inside the word (compile-time constant at every call)
    uint4 e[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) e[p] = make_uint4(w[p], 0u, 0u, 0u);
    if constexpr (EST == 1)
        select_2of4_approx(Row<NM_DT_BF16>::get(e[0], half), Row<NM_DT_BF16>::get(e[1], half), Row<NM_DT_BF16>::get(e[2], half),
                           Row<NM_DT_BF16>::get(e[3], half), word1, word2, v0, v1, nib);
    else
        select_2of4<NM_DT_BF16>(Key<NM_DT_BF16>::make(e[0], half, 0), Key<NM_DT_BF16>::make(e[1], half, 1), Key<NM_DT_BF16>::make(e[2], half, 2),
                                Key<NM_DT_BF16>::make(e[3], half, 3), word1, v0, v1, nib);
}

template <bool HI0>
__device__ __forceinline__ void philox_call(uint64_t ctr, uint32_t stream_id, uint32_t domain, uint32_t key0, uint32_t key1, uint32_t (&w4)[4])
{
    if constexpr (HI0) philox4x32_10_uniform_c123((uint32_t)ctr, 0u, stream_id, domain, key0, key1, w4);
    else philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), stream_id, domain, key0, key1, w4);
}

template <int EST, bool HI0>
__device__ __forceinline__ void prune_grid(uint32_t *tile, int64_t *offs, const uint16_t *__restrict__ g, const GridGeom &gg, bool cl, int64_t n_groups,
                                           uint32_t key0, uint32_t key1, uint32_t stream_id, uint16_t *__restrict__ vals,
                                           uint16_t *__restrict__ meta, int64_t bx, int by)
{
    const int64_t r0 = bx * TILE_ROWS;
    const int c0 = by * TILE_COLS, O = gg.C;
    load_tile(tile, offs, g, gg, cl, r0, c0);

    const int tid = threadIdx.x, cq = tid & 15, gi = tid >> 4;          // four columns 4cq .. 4cq+3 of token group gi of the tile
    const int64_t G = r0 / 16 + gi;
    const int col = c0 + 4 * cq;
    uint32_t kept[4][4], md[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint2 row[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) row[p] = *(const uint2 *)(tile + (16 * gi + 4 * b + p) * TILE_LD + 2 * cq);
        const uint64_t blk0 = (uint64_t)(G * 4 + b) * (uint64_t)O + (uint64_t)col;
        uint32_t words[EST == 1 ? 8 : 4];
#pragma unroll
        for (int q = 0; q < (EST == 1 ? 2 : 1); ++q) {
            uint32_t w4[4];
            philox_call<HI0>((blk0 >> (EST == 1 ? 1 : 2)) + q, stream_id, EST == 1 ? 1u : 0u, key0, key1, w4);
#pragma unroll
            for (int j = 0; j < 4; ++j) words[4 * q + j] = w4[j];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t w[4] = {c < 2 ? row[0].x : row[0].y, c < 2 ? row[1].x : row[1].y, c < 2 ? row[2].x : row[2].y, c < 2 ? row[3].x : row[3].y};
            float v0, v1; uint32_t nib;
            select_quad_bf16<EST>(w, c & 1, EST == 1 ? words[2 * c] : words[c], EST == 1 ? words[2 * c + 1] : 0u, v0, v1, nib);
            kept[c][b] = pack_bf16_rne(v0, v1);
            md[c] |= nib << (4 * b);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the wave's own 64 tile rows (4 groups) become its exchange area: column l of group k at slot 64k + (l with its low two bits
    // swizzled by the next two)
    const int lane = tid & 63;
    char *xw = (char *)(tile + (tid >> 6) * 64 * TILE_LD);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < 4; ++c)
        *(uint4 *)(xw + (64 * (gi & 3) + 4 * cq + (c ^ (cq & 3))) * 16) = make_uint4(kept[c][0], kept[c][1], kept[c][2], kept[c][3]);
    __builtin_amdgcn_wave_barrier();
    const int64_t Gw = r0 / 16 + (tid >> 6) * 4;
    const int slot = (lane & ~3) | ((lane & 3) ^ ((lane >> 2) & 3));
    if (c0 + lane < O) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (Gw + k < n_groups) *(uint4 *)(vals + ((Gw + k) * O + c0 + lane) * 8) = *(const uint4 *)(xw + (64 * k + slot) * 16);
    }
    if (col < O && G < n_groups) *(uint2 *)(meta + G * O + col) = make_uint2(md[0] | (md[1] << 16), md[2] | (md[3] << 16));
}

template <int EST, bool HI0>
__device__ __forceinline__ void prune_grid_q8(uint32_t *tile, int64_t *offs, const uint16_t *__restrict__ g, const GridGeom &gg, bool cl, int64_t n_groups,
                                              uint32_t key0, uint32_t key1, uint32_t stream_id, const LayerScale &ls,
                                              uint8_t *__restrict__ vals8, uint32_t *__restrict__ meta32, int64_t bx, int by)
{
    const int64_t r0 = bx * TILE_ROWS;
    const int c0 = by * TILE_COLS, O = gg.C;
    const uint4 peaks = layer_peaks(ls);
    load_tile(tile, offs, g, gg, cl, r0, c0);
    const float scale = layer_scale(ls, peaks, bx == 0 && by == 0);

    const int tid = threadIdx.x, cp = tid & 31, gi = tid >> 5;          // columns 2cp, 2cp+1 of token group gi (8 groups in the tile)
    const bool odd = cp & 1;
    const int64_t G = r0 / 32 + gi;
    const int col = c0 + 2 * cp;
    uint32_t kept[2][4] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, md[2] = {0u, 0u};
    static_for<8>([&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
        uint32_t w[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) w[p] = tile[(32 * gi + 4 * b + p) * TILE_LD + cp];
        const uint64_t blk0 = (uint64_t)(G * 8 + b) * (uint64_t)O + (uint64_t)(col & ~3);      // first of the pair's four columns
        uint32_t sel[4], rnd[2];
        uint32_t w4[4];
        if constexpr (EST == 1) {
            philox_call<HI0>((blk0 >> 1) + (odd ? 1 : 0), stream_id, 1u, key0, key1, sel);     // two words for each of its two columns
            philox_call<HI0>(blk0 >> 2, stream_id, 2u, key0, key1, w4);
            rnd[0] = odd ? w4[2] : w4[0]; rnd[1] = odd ? w4[3] : w4[1];
        } else {
            const uint64_t ctr = blk0 >> 2;
            philox4x32_10((uint32_t)ctr, HI0 ? 0u : (uint32_t)(ctr >> 32), stream_id, odd ? 2u : 0u, key0, key1, w4);
            const uint32_t r0w = swap_pair(odd ? w4[0] : w4[2]), r1w = swap_pair(odd ? w4[1] : w4[3]);
            sel[0] = odd ? r0w : w4[0]; sel[2] = odd ? r1w : w4[1];
            rnd[0] = odd ? w4[2] : r0w; rnd[1] = odd ? w4[3] : r1w;
            sel[1] = sel[3] = 0u;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float v0, v1; uint32_t nib;
            select_quad_bf16<EST>(w, c, sel[2 * c], sel[2 * c + 1], v0, v1, nib);
            kept[c][b / 2] = sr_e5m2_into<2 * (b & 1)>(kept[c][b / 2], v0 * scale, rnd[c] << 16);
            kept[c][b / 2] = sr_e5m2_into<2 * (b & 1) + 1>(kept[c][b / 2], v1 * scale, rnd[c] & 0xffff0000u);
            md[c] |= nib << (4 * b);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
    // exchange through the wave's own 64 tile rows (2 groups): column l of group k at slot 64k + (l with bit 0 swizzled by bit 2)
    const int lane = tid & 63;
    char *xw = (char *)(tile + (tid >> 6) * 64 * TILE_LD);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < 2; ++c)
        *(uint4 *)(xw + (64 * (gi & 1) + 2 * cp + (c ^ ((cp >> 1) & 1))) * 16) = make_uint4(kept[c][0], kept[c][1], kept[c][2], kept[c][3]);
    __builtin_amdgcn_wave_barrier();
    const int64_t Gw = r0 / 32 + (tid >> 6) * 2;
    const int slot = (lane & ~1) | ((lane & 1) ^ ((lane >> 2) & 1));
    if (c0 + lane < O) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (Gw + k < n_groups) *(uint4 *)(vals8 + ((Gw + k) * O + c0 + lane) * 16) = *(const uint4 *)(xw + (64 * k + slot) * 16);
    }
    if (col < O && G < n_groups) *(uint2 *)(meta32 + G * O + col) = make_uint2(md[0], md[1]);
}

struct PackTask { const uint16_t *x; GridGeom gg; bool cl; int64_t margin, out_rows; LayerScale ls; void *out; int64_t rows, blocks; };
struct PruneTask { const uint16_t *g; GridGeom gg; bool cl; int64_t n_groups; LayerScale ls; void *vals, *meta; int64_t rows, blocks; };

// `rows` workgroups along the grid's rows (fastest) and the rest along the channels, for either task
template <bool Q8, int EST, bool HI0>
__global__ __launch_bounds__(256) void grid_kernel(PackTask a, PruneTask b, uint32_t key0, uint32_t key1, uint32_t stream_id)
{
    __shared__ __attribute__((aligned(16))) uint32_t tile[TILE_ROWS * TILE_LD];
    __shared__ int64_t offs[TILE_ROWS];
    // workgroup n is a pack where the running share of packs, n * blocks / total, steps at n+1
    const int64_t total = a.blocks + b.blocks, n = blockIdx.x, packs = n * a.blocks / total;
    if ((n + 1) * a.blocks / total != packs) {
        grid_pack<Q8>(tile, offs, a.x, a.gg, a.cl, a.margin, a.out_rows, a.ls, a.out, packs % a.rows, (int)(packs / a.rows));
    } else {
        const int64_t p = n - packs;
        if constexpr (Q8)
            prune_grid_q8<EST, HI0>(tile, offs, b.g, b.gg, b.cl, b.n_groups, key0, key1, stream_id, b.ls, (uint8_t *)b.vals, (uint32_t *)b.meta,
                                    p % b.rows, (int)(p / b.rows));
        else
            prune_grid<EST, HI0>(tile, offs, b.g, b.gg, b.cl, b.n_groups, key0, key1, stream_id, (uint16_t *)b.vals, (uint16_t *)b.meta,
                                 p % b.rows, (int)(p / b.rows));
    }
}

// x, margin, out_rows, sx, x_out: the activations' rows [-margin, out_rows - margin), as bf16 (sx == nullptr) or e4m3.
// est: 0 optimal MVUE 2:4, 1 approx-MVUE 2:4; T: the gradient's grid rows rounded up to whole groups (16 tokens, or 32 with sg: 8-bit)
hipError_t launch_grid(const ConvShape &cs, const void *x, int64_t margin, int64_t out_rows, const LayerScale *sx, void *x_out, int est,
                       const void *gy, int64_t T, uint64_t seed, uint32_t stream_id, const LayerScale *sg, void *vals, void *meta, hipStream_t st)
{
    const bool q8 = sg != nullptr;
    PackTask a{(const uint16_t *)x, grid_geom(cs, cs.C), cs.x_channels_last, margin, out_rows, q8 ? *sx : LayerScale{}, x_out, (out_rows + TILE_ROWS - 1) / TILE_ROWS, 0};
    PruneTask b{(const uint16_t *)gy, grid_geom(cs, cs.O), cs.g_channels_last, T / (q8 ? 32 : 16), q8 ? *sg : LayerScale{}, vals, meta, (T + TILE_ROWS - 1) / TILE_ROWS, 0};
    a.blocks = a.rows * ((cs.C + TILE_COLS - 1) / TILE_COLS);
    b.blocks = b.rows * ((cs.O + TILE_COLS - 1) / TILE_COLS);
    if (a.blocks + b.blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    // call indices are at most T*O/8 + 1 (approx-MVUE; a quarter block row less otherwise)
    const bool hi0 = (uint64_t)T * (uint64_t)cs.O <= ((uint64_t)1 << 34);
    const dim3 grid((unsigned)(a.blocks + b.blocks));
#define NM_GRID(Q8, EST, HI0) hipLaunchKernelGGL((grid_kernel<Q8, EST, HI0>), grid, dim3(256), 0, st, a, b, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id)
#define NM_GRID2(Q8, EST) do { if (hi0) NM_GRID(Q8, EST, true); else NM_GRID(Q8, EST, false); } while (0)
    if (q8) { if (est == 1) NM_GRID2(true, 1); else NM_GRID2(true, 0); }
    else { if (est == 1) NM_GRID2(false, 1); else NM_GRID2(false, 0); }
#undef NM_GRID2
#undef NM_GRID
    return hipGetLastError();
}

}  // namespace nm
