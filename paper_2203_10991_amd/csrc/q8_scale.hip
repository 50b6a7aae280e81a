// Per-tensor scale and the activations' 8-bit cast of the 8-bit path (Sec. 5, 8-bit rows; the paper fixes no scale
// rule).  One power-of-two scale per tensor from its current maximum magnitude: the largest s = 2^e with
// s * max|t| <= top, e kept in [-126, 126] so that s and 1/s are normal numbers, s = 1 for an all-zero tensor or a
// maximum that is not finite.  The scale never visits the host: it is written to a 4-float record in device memory
//     rec[0] = s,  rec[1] = 1/s,  rec[2] = bit pattern of max|t|,  rec[3] = 0
// which the 8-bit prune, the cast below and the 8-bit update GEMM read there.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "nm_internal.h"
#include "q8_scale.h"

namespace nm {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// (a fill kernel, not a memset: safe to record into a HIP graph)
__global__ void q8_scale_begin_kernel(float *rec)
{
    if (threadIdx.x < 4) ((uint32_t *)rec)[threadIdx.x] = 0u;
}

// max over the bit patterns of |t|: they order like the magnitudes, with infinity and every NaN on top (the maximum does
// not depend on the order of the atomics: the result is reproducible), and the scale from it, in one launch.
// Bound: HBM, one read of the tensor.  What it took instead was the atomics: one per wave on a single address, about 10 ns
// each one after the other (16384 of them: 155 us for a 20 MB tensor that streams in 4 us).  So a workgroup of 1024 threads
// takes 128 KB or more with four independent 16-byte loads in flight per thread, reduces through LDS, and touches the record
// only when its maximum is above what is there; a ticket in rec[3] lets the last workgroup write the scale, which a launch of
// its own did before.  At most one workgroup per CU: the tickets queue up on one address as well (a sweep with 128 / 256 / 512 /
// 1024 workgroups: 12608 x 3072 22 / 22 / 36 / 50 us, 32768 x 28672 350 / 311 / 322 / 343 us; and with 16 instead of 128 KB per
// workgroup 4096 x 1024 takes 12-17 us instead of 10).
// A contiguous tensor is one row of R * C elements: the 64-bit division of a piece's number by the row length, once per
// 16 bytes, cost more instructions than everything else in the loop.  Strided rows of at most 1024 pieces go several to a trip, each on
// the smallest power of two of threads that holds it, four trips' loads in flight (with a row per trip 802816 x 64 bf16 at a
// stride of 128 took 1077 us on eight threads of every workgroup; now 23; 50176 x 256 at 512 51 -> 11, 32768 x 8192 at 8200 110 -> 96).
// Measured, launches included, before -> after: 12608 x 768 bf16 192 -> 11 us, 32768 x 28672 398 -> 312 us (6.0 TB/s).
constexpr int AMAX_THREADS = 1024, AMAX_BLOCKS = 256, AMAX_UNROLL = 4;
static_assert(AMAX_BLOCKS <= LAYER_PEAKS, "a word for every workgroup");
constexpr int AMAX_PIECES = 8 * AMAX_THREADS;         // 16-byte pieces a workgroup takes at least: 128 KB (of a strided row that is longer than a trip: one row)

template <int DT> __device__ __forceinline__ uint32_t amax_piece(uint32_t m, const u32x4_t &v)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (DT == NM_DT_F32) m = max(m, v[j] & 0x7fffffffu);
        else { m = max(m, (v[j] << 16) & 0x7fff0000u); m = max(m, v[j] & 0x7fff0000u); }
    }
    return m;
}

// one tensor of a launch: R rows of C elements at a stride of ld, handled by `blocks` workgroups.  row_shift >= 0: rows of at most
// 1024 pieces, 2^row_shift threads to a row; -1: workgroups share rows or take them one by one
struct AmaxArg { const void *t; int64_t R, C, ld; float top; float *rec; int blocks, row_shift; };

// (a launch takes one tensor, or the two of a layer: workgroups [0, a.blocks) the first, the others the second)
// PEAKS: a workgroup leaves its maximum in rec[bid] (a word each) and the kernels behind this one find the scale from those (layer_scale): no record
// to clear before and no tickets.  A layer's calls run so: with the records cleared by a launch before and the last workgroup's
// scale, the 8-bit 14 x 14 convolution layer took 78.4 us (now 69.6) and the 8-bit linear layer 12608 x 3072 -> 768 241.6 (now 235.8).
template <int DT, bool PEAKS>
__global__ __launch_bounds__(AMAX_THREADS) void q8_amax_kernel(AmaxArg a, AmaxArg b)
{
    const bool second = (int)blockIdx.x >= a.blocks;
    const int64_t bid = second ? blockIdx.x - a.blocks : blockIdx.x, n_blocks = second ? b.blocks : a.blocks;
    const void *t_ = second ? b.t : a.t;
    const int64_t R = second ? b.R : a.R, C = second ? b.C : a.C, ld = second ? b.ld : a.ld;
    const float top = second ? b.top : a.top;
    float *rec = second ? b.rec : a.rec;
    constexpr int VEC = DT == NM_DT_F32 ? 4 : 8, ESZ = DT == NM_DT_F32 ? 4 : 2;
    const int row_shift = second ? b.row_shift : a.row_shift;
    const int64_t cpr = C / VEC;
    uint32_t m = 0;
    // `split` workgroups share a row when there are fewer rows than workgroups
    const int64_t split = R >= n_blocks ? 1 : n_blocks / R;
    const int64_t part = bid % split;
    if (row_shift >= 0) {
        const int64_t step = n_blocks * (AMAX_THREADS >> row_shift), piece = threadIdx.x & ((1 << row_shift) - 1);
        if (piece < cpr) {
            int64_t r = bid * (AMAX_THREADS >> row_shift) + (threadIdx.x >> row_shift);
            const char *at = (const char *)t_ + (r * ld + piece * VEC) * ESZ;
            const int64_t step_bytes = step * ld * ESZ;
            for (; r + (AMAX_UNROLL - 1) * step < R; r += AMAX_UNROLL * step, at += AMAX_UNROLL * step_bytes) {
                u32x4_t v[AMAX_UNROLL];
#pragma unroll
                for (int k = 0; k < AMAX_UNROLL; ++k) v[k] = *(const u32x4_t *)(at + k * step_bytes);
#pragma unroll
                for (int k = 0; k < AMAX_UNROLL; ++k) m = amax_piece<DT>(m, v[k]);
            }
            for (; r < R; r += step, at += step_bytes) m = amax_piece<DT>(m, *(const u32x4_t *)at);
        }
    } else
    for (int64_t r = bid / split; r < R; r += n_blocks / split) {
        const u32x4_t *row = (const u32x4_t *)((const char *)t_ + r * ld * ESZ);
        int64_t i = part * AMAX_THREADS + threadIdx.x;
        const int64_t step = split * AMAX_THREADS;
        for (; i + (AMAX_UNROLL - 1) * step < cpr; i += AMAX_UNROLL * step) {
            u32x4_t v[AMAX_UNROLL];
#pragma unroll
            for (int k = 0; k < AMAX_UNROLL; ++k) v[k] = row[i + k * step];
#pragma unroll
            for (int k = 0; k < AMAX_UNROLL; ++k) m = amax_piece<DT>(m, v[k]);
        }
        for (; i < cpr; i += step) m = amax_piece<DT>(m, row[i]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    __shared__ uint32_t wave_max[AMAX_THREADS / 64];
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int w = 1; w < AMAX_THREADS / 64; ++w) m = max(m, wave_max[w]);
    if constexpr (PEAKS) {
        ((uint32_t *)rec)[bid] = m;
        return;
    }
    uint32_t *top_bits = (uint32_t *)rec + 2, *ticket = (uint32_t *)rec + 3;
    if (m > __hip_atomic_load(top_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        const uint32_t before = __hip_atomic_fetch_max(top_bits, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : : "v"(before));                        // (returning form: the wait below covers it)
    }
    // Every access to the record is a device-scope atomic, done where all XCDs meet, so it is enough that this workgroup's
    // maximum has been performed (the wait) before its ticket: a release or acquire at this scope would write back and
    // invalidate the XCD's L2, once per workgroup.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (__hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint32_t)n_blocks - 1) return;
    float s, inv;
    scale_of_max(__hip_atomic_load(top_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), top, s, inv);
    rec[0] = s;
    rec[1] = inv;
    *ticket = 0;
}

// an empty tensor: scale 1, every word of the record written
__global__ void q8_scale_empty_kernel(float *rec)
{
    if (threadIdx.x < 4) rec[threadIdx.x] = threadIdx.x < 2 ? 1.0f : 0.0f;
}

static AmaxArg amax_arg(int dt, const void *t, int64_t R, int64_t C, int64_t ld, float top, float *rec, int most_blocks)
{
    if (ld == C) { C *= R; ld = C; R = 1; }
    const int64_t cpr = C / (dt == NM_DT_F32 ? 4 : 8);
    if (R > 1 && cpr <= AMAX_THREADS) {
        int shift = 0;
        while (((int64_t)1 << shift) < cpr) ++shift;
        const int64_t rows = AMAX_PIECES >> shift;                             // rows of a workgroup's least share
        return AmaxArg{t, R, C, ld, top, rec, (int)std::min<int64_t>(most_blocks, (R + rows - 1) / rows), shift};
    }
    const int64_t per_row = (cpr + AMAX_PIECES - 1) / AMAX_PIECES;            // workgroups that a row's pieces fill
    const int64_t blocks = R >= most_blocks ? most_blocks : R * std::min<int64_t>(per_row, most_blocks / R);
    return AmaxArg{t, R, C, ld, top, rec, (int)blocks, -1};
}

hipError_t launch_q8_scale(int dt, const void *t, int64_t R, int64_t C, int64_t ld, float top, float *rec, hipStream_t st)
{
    if (R == 0 || C == 0) {
        hipLaunchKernelGGL(q8_scale_empty_kernel, dim3(1), dim3(64), 0, st, rec);
        return hipGetLastError();
    }
    const AmaxArg a = amax_arg(dt, t, R, C, ld, top, rec, AMAX_BLOCKS);
    hipLaunchKernelGGL(q8_scale_begin_kernel, dim3(1), dim3(64), 0, st, rec);
    if (dt == NM_DT_F32) hipLaunchKernelGGL((q8_amax_kernel<NM_DT_F32, false>), dim3((unsigned)a.blocks), dim3(AMAX_THREADS), 0, st, a, AmaxArg{});
    else hipLaunchKernelGGL((q8_amax_kernel<NM_DT_BF16, false>), dim3((unsigned)a.blocks), dim3(AMAX_THREADS), 0, st, a, AmaxArg{});
    return hipGetLastError();
}

hipError_t launch_layer_peaks(const void *t0, int64_t R0, int64_t C0, int64_t ld0, LayerScale &s0, const void *t1, int64_t R1, int64_t C1, int64_t ld1,
                              LayerScale &s1, hipStream_t st)
{
    const int64_t n0 = R0 * C0, n1 = R1 * C1;                    // the workgroups are dealt by size
    const int most0 = (int)std::max<int64_t>(1, std::min<int64_t>(AMAX_BLOCKS - 1, (int64_t)((double)AMAX_BLOCKS * (double)n0 / (double)(n0 + n1))));
    const AmaxArg a = amax_arg(NM_DT_BF16, t0, R0, C0, ld0, s0.top, (float *)s0.peaks, most0);
    const AmaxArg b = amax_arg(NM_DT_BF16, t1, R1, C1, ld1, s1.top, (float *)s1.peaks, AMAX_BLOCKS - most0);
    s0.n = a.blocks; s1.n = b.blocks;
    hipLaunchKernelGGL((q8_amax_kernel<NM_DT_BF16, true>), dim3((unsigned)(a.blocks + b.blocks)), dim3(AMAX_THREADS), 0, st, a, b);
    return hipGetLastError();
}

// binary32 -> e4m3 (OCP), round to nearest even, magnitudes beyond 448 saturate: the hardware conversion after a
// clamp (it would otherwise produce the format's NaN where this cast saturates).  Four values per call pair.
__device__ __forceinline__ uint32_t pack4_e4m3(float a, float b, float c, float d)
{
    a = __builtin_amdgcn_fmed3f(a, -448.0f, 448.0f); b = __builtin_amdgcn_fmed3f(b, -448.0f, 448.0f);
    c = __builtin_amdgcn_fmed3f(c, -448.0f, 448.0f); d = __builtin_amdgcn_fmed3f(d, -448.0f, 448.0f);
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    return (uint32_t)w;
}

// one thread = 16 consecutive elements of a row -> one 16-byte store; rows past the R of h are zero codes
// LAYER: the scale from the maxima of ls; otherwise rec's
template <int DT, bool LAYER = false>
__global__ __launch_bounds__(256) void cast_e4m3_kernel(const void *__restrict__ h_, int64_t R, int64_t C, int64_t ld, const float *__restrict__ rec,
                                                       LayerScale ls, uint8_t *__restrict__ h8, int64_t ld8, int64_t out_rows)
{
    [[maybe_unused]] uint4 peaks;
    if constexpr (LAYER) peaks = layer_peaks(ls);
    const int64_t cpr = C / 16, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t r = i / cpr, c = (i - r * cpr) * 16;
    constexpr int PIECES = DT == NM_DT_F32 ? 4 : 2;
    u32x4_t v[PIECES];
#pragma unroll
    for (int j = 0; j < PIECES; ++j) v[j] = u32x4_t{0u, 0u, 0u, 0u};
    if (i < out_rows * cpr && r < R) {
        const u32x4_t *src = (const u32x4_t *)((const char *)h_ + (r * ld + c) * (DT == NM_DT_F32 ? 4 : 2));
#pragma unroll
        for (int j = 0; j < PIECES; ++j) v[j] = src[j];
    }
    float s;
    if constexpr (LAYER) s = layer_scale(ls, peaks, blockIdx.x == 0);
    else s = rec[0];
    if (i >= out_rows * cpr) return;
    u32x4_t o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if constexpr (DT == NM_DT_F32) x[k] = __uint_as_float(v[j][k]);
            else { const uint32_t w = v[j / 2][2 * (j % 2) + k / 2]; x[k] = __uint_as_float(k % 2 ? w & 0xffff0000u : w << 16); }
        o[j] = pack4_e4m3(x[0] * s, x[1] * s, x[2] * s, x[3] * s);
    }
    *(u32x4_t *)(h8 + r * ld8 + c) = r < R ? o : u32x4_t{0u, 0u, 0u, 0u};
}

// a layer's activations (bf16), rows past the R of h up to out_rows as zeros
hipError_t launch_cast_e4m3_layer(const void *h, int64_t R, int64_t C, int64_t ld, const LayerScale &ls, uint8_t *h8, int64_t ld8, int64_t out_rows,
                                  hipStream_t st)
{
    const int64_t blocks = (out_rows * (C / 16) + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((cast_e4m3_kernel<NM_DT_BF16, true>), dim3((unsigned)blocks), dim3(256), 0, st, h, R, C, ld, (const float *)nullptr, ls, h8, ld8, out_rows);
    return hipGetLastError();
}

hipError_t launch_cast_e4m3(int dt, const void *h, int64_t R, int64_t C, int64_t ld, const float *rec, uint8_t *h8, int64_t ld8,
                            hipStream_t st)
{
    const int64_t threads = R * (C / 16);
    if (threads == 0) return hipSuccess;
    const int64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    if (dt == NM_DT_F32) hipLaunchKernelGGL(cast_e4m3_kernel<NM_DT_F32>, dim3((unsigned)blocks), dim3(256), 0, st, h, R, C, ld, rec, LayerScale{}, h8, ld8, R);
    else hipLaunchKernelGGL(cast_e4m3_kernel<NM_DT_BF16>, dim3((unsigned)blocks), dim3(256), 0, st, h, R, C, ld, rec, LayerScale{}, h8, ld8, R);
    return hipGetLastError();
}

}  // namespace nm
