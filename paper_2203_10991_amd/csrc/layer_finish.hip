// The second pass of a layer's update GEMM: the slabs' partial sums become the weight gradient in the layout and type the
// layer stores its weight in.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "smfmac_common.h"       // alpha_of
#include "prune_common.h"        // pack_bf16_rne

namespace nm {

// Convolution: dW[o][c][tap] (bf16) = alpha * sum_z part[z][o][tap][c].  A workgroup takes one output channel and CW input
// channels: R threads share a float4 of the partial sums (as in splitk_reduce_kernel: thread r sums slabs r, r+R, ... in
// order, a fixed tree combines them), the results turn through LDS, and the CW x taps values leave contiguous.
// Bound: launch latency and one read of the partial sums.  A sum of up to 11 slabs is one chain, of up to 63 eight, beyond that 16 (the order of the
// additions depends on the slab count only).  Large layers have a thread to a sum, all its chains side by side, in workgroups 64 channels
// wide; others would leave the GPU idle so and have a thread to a chain, in workgroups 32 (16) channels wide.  Partial sums in the caches, thread a sum /
// thread a chain, us: 64 x 64 x 9 of 46 slabs 6.5 / 4.4, 128 x 128 x 9 of 24 4.7 / 4.8, of 46 7.7 / 6.6, 256 x 128 x 9 of 12 5.3 / 5.9, of 46 10.6 / 11.3, 256 x 256 x 9 of
// 24 10.1 / 12.5, 96 x 256 x 1 in its layer 7.1 / 4.2, 256 x 256 x 1 of 24 4.0 / 7.2; 64 x 64 x 9 of 254 15.5 / 8.8, 128 x 256 x 9 of 96 17.6 / 19.7, 256 x 128 x 1 in its
// layer 8.8 / 6.9.
template <int R, int CHAINS, int CW, int NT>
__global__ __launch_bounds__(NT) void finish_conv_kernel(const float *__restrict__ part, int slabs, int64_t slab_stride, uint16_t *__restrict__ dW,
                                                         int C, int taps, AlphaArg al)
{
    __shared__ uint16_t turned[CW * 32];                                 // [channel][tap]
    const float alpha = alpha_of(al);
    const int64_t o = blockIdx.x;
    const int c0 = (int)blockIdx.y * CW, cols = min(CW, C - c0), q4 = cols / 4;
    const float *src = part + o * (int64_t)taps * C + c0;
    const int r = threadIdx.x % R, tasks = taps * q4;
    for (int t0 = 0; t0 < tasks; t0 += NT / R) {
        const int t = t0 + threadIdx.x / R;
        const bool valid = t < tasks;
        const int tap = valid ? t / q4 : 0, c = valid ? (t % q4) * 4 : 0;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (valid) s = sum_of_slabs<R, CHAINS, 4>(src + (int64_t)tap * C + c, r, slabs, slab_stride);
        s = sum_of_threads<R>(s);
        if (valid && r == 0) {
            const uint32_t a = pack_bf16_rne(s.x * alpha, s.y * alpha), b = pack_bf16_rne(s.z * alpha, s.w * alpha);
            turned[(c + 0) * taps + tap] = (uint16_t)a; turned[(c + 1) * taps + tap] = (uint16_t)(a >> 16);
            turned[(c + 2) * taps + tap] = (uint16_t)b; turned[(c + 3) * taps + tap] = (uint16_t)(b >> 16);
        }
    }
    __syncthreads();
    uint32_t *dst = (uint32_t *)(dW + (o * C + c0) * taps);              // (c0 and C are multiples of 8: whole words)
    for (int i = threadIdx.x; i < cols * taps / 2; i += NT) dst[i] = *(const uint32_t *)&turned[2 * i];
}

hipError_t launch_finish_conv(const float *part, int slabs, void *dW, int64_t O, int C, int taps, AlphaArg alpha, hipStream_t st)
{
#define NM_FINISH(R, CHAINS, CW, NT)                                                                                                              \
    hipLaunchKernelGGL((finish_conv_kernel<R, CHAINS, CW, NT>), dim3((unsigned)O, (unsigned)((C + CW - 1) / CW)), dim3(NT), 0, st, part, slabs,    \
                       O * (int64_t)taps * C, (uint16_t *)dW, C, taps, alpha)
    const bool large = O * C > 128 * 128 && O * C * taps >= 65536;
    if (slabs >= 64) { if (large) NM_FINISH(1, 16, 64, 256); else NM_FINISH(16, 1, 16, 576); }
    else if (slabs >= 12) { if (large) NM_FINISH(1, 8, 64, 256); else NM_FINISH(8, 1, 32, 576); }
    else NM_FINISH(1, 1, 64, 256);
#undef NM_FINISH
    return hipGetLastError();
}

// Linear: dW[o][i] (bf16) = alpha * sum_z part[z][o][i], and beside it -- the first db_blocks workgroups -- the bias gradient
// db[o] (bf16) = the sum of the token groups' column sums csum[G][o].  The sums of dW run as in splitk_reduce_kernel (R threads
// per float4); a column's groups are summed by 64 threads, each a strided share in order, and a fixed tree over LDS.
// Bound: launch latency and one read of the partial sums.  Sum, conversion and bias were three to five launches.  The bias
// workgroups walk a chain of loads (1024 groups: 16 per thread), so they start first and keep four in flight: 16384 x 4096 x 1024
// in four slabs 26 -> 18 us.
constexpr int DB_COLS = 16;                                              // columns of a bias workgroup: 4 float4 x 64 groups in flight
template <int R, int CHAINS>
__global__ __launch_bounds__(256) void finish_linear_kernel(const float *__restrict__ part, int slabs, int64_t O, int64_t I, uint16_t *__restrict__ dW,
                                                            AlphaArg al, int db_blocks, const float *__restrict__ csum, int64_t groups,
                                                            uint16_t *__restrict__ db)
{
    __shared__ float4 sums[256];
    if ((int)blockIdx.x >= db_blocks) {
        const float alpha = alpha_of(al);
        const int64_t n4 = O * I / 4, idx = (int64_t)(blockIdx.x - db_blocks) * (256 / R) + threadIdx.x / R;       // (I % 8 == 0: rows are whole float4s)
        const int r = threadIdx.x % R;
        const bool valid = idx < n4;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (valid) s = sum_of_slabs<R, CHAINS>(part + idx * 4, r, slabs, O * I);
        s = sum_of_threads<R>(s);
        if (valid && r == 0) *(uint2 *)(dW + idx * 4) = make_uint2(pack_bf16_rne(s.x * alpha, s.y * alpha), pack_bf16_rne(s.z * alpha, s.w * alpha));
        return;
    }
    const int64_t c0 = (int64_t)blockIdx.x * DB_COLS + (threadIdx.x & 3) * 4;
    const int g = threadIdx.x >> 2;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c0 < O)
#pragma unroll 4
        for (int64_t G = g; G < groups; G += 64) {
            const float4 v = *(const float4 *)(csum + G * O + c0);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
    sums[threadIdx.x] = s;
    for (int d = 32; d >= 1; d >>= 1) {
        __syncthreads();
        if (g < d) {
            const float4 v = sums[threadIdx.x + 4 * d];
            float4 &m = sums[threadIdx.x];
            m.x += v.x; m.y += v.y; m.z += v.z; m.w += v.w;
        }
    }
    if (g == 0 && c0 < O) {
        const float4 m = sums[threadIdx.x];
        *(uint2 *)(db + c0) = make_uint2(pack_bf16_rne(m.x, m.y), pack_bf16_rne(m.z, m.w));
    }
}

hipError_t launch_finish_linear(const float *part, int slabs, int64_t O, int64_t I, void *dW, AlphaArg alpha, const float *csum, int64_t groups,
                                void *db, hipStream_t st)
{
    const SlabSum form = slab_sum_form(O * I / 4, slabs);
    const int R = form == SlabSum::shared ? 8 : 1;
    const int64_t dw_blocks = (O * I / 4 + 256 / R - 1) / (256 / R), db_blocks = db ? (O + DB_COLS - 1) / DB_COLS : 0;
    if (dw_blocks + db_blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(dw_blocks + db_blocks));
#define NM_FINISH(R, CHAINS)                                                                                                                  \
    hipLaunchKernelGGL((finish_linear_kernel<R, CHAINS>), grid, dim3(256), 0, st, part, slabs, O, I, (uint16_t *)dW, alpha, (int)db_blocks, csum, \
                       groups, (uint16_t *)db)
    switch (form) {
    case SlabSum::one_chain: NM_FINISH(1, 1); break;
    case SlabSum::eight_chains: NM_FINISH(1, 8); break;
    case SlabSum::shared: NM_FINISH(8, 1); break;
    }
#undef NM_FINISH
    return hipGetLastError();
}

// rows [0, rows) of h (C columns, row stride ld, bf16) and zeros up to out_rows, contiguous
__global__ __launch_bounds__(256) void pad_rows_kernel(const uint16_t *__restrict__ h, int64_t rows, int64_t C, int64_t ld, uint16_t *__restrict__ out, int64_t out_rows)
{
    const int64_t cpr = C / 8, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= out_rows * cpr) return;
    const int64_t r = i / cpr, c = (i - r * cpr) * 8;
    *(uint4 *)(out + r * C + c) = r < rows ? *(const uint4 *)(h + r * ld + c) : make_uint4(0u, 0u, 0u, 0u);
}

hipError_t launch_pad_rows(const void *h, int64_t rows, int64_t C, int64_t ld, void *out, int64_t out_rows, hipStream_t st)
{
    const int64_t blocks = (out_rows * (C / 8) + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(pad_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const uint16_t *)h, rows, C, ld, (uint16_t *)out, out_rows);
    return hipGetLastError();
}

}  // namespace nm
