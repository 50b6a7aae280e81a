// The second pass of a layer's update GEMM: the slabs' partial sums become the weight gradient in the layout and type the
// layer stores its weight in.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "smfmac_common.h"       // alpha_of
#include "prune_common.h"        // pack_bf16_rne

namespace nm {

// Convolution: dW[o][c][tap] (bf16) = alpha * sum_z part[z][o][tap][c].  A workgroup takes one output channel and 64 input
// channels: R threads share a float4 of the partial sums (as in splitk_reduce_kernel: thread r sums slabs r, r+R, ... in
// order, a fixed tree combines them), the results turn through LDS, and the 64 x taps values leave contiguous.
// Bound: launch latency and one read of the partial sums.  Summing, permuting and converting were three launches and
// 15-20 us on ResNet-50's layers; this is one of 6-10 us.
// With many slabs (R = 8) the workgroup has 1024 threads: 128 of the up to 16 x taps sums run at a time.
template <int R>
__global__ __launch_bounds__(R == 8 ? 1024 : 256) void finish_conv_kernel(const float *__restrict__ part, int slabs, int64_t slab_stride, uint16_t *__restrict__ dW,
                                                          int C, int taps, AlphaArg al)
{
    __shared__ uint16_t turned[64 * 32];                                 // [channel][tap]
    constexpr int NT = R == 8 ? 1024 : 256;
    const float alpha = alpha_of(al);
    const int64_t o = blockIdx.x;
    const int c0 = (int)blockIdx.y * 64, cols = min(64, C - c0), q4 = cols / 4;
    const float *src = part + o * (int64_t)taps * C + c0;
    const int r = threadIdx.x % R, tasks = taps * q4;
    for (int t0 = 0; t0 < tasks; t0 += NT / R) {
        const int t = t0 + threadIdx.x / R;
        const bool valid = t < tasks;
        const int tap = valid ? t / q4 : 0, c = valid ? (t % q4) * 4 : 0;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (valid)
            for (int z = r; z < slabs; z += R) {
                const float4 v = *(const float4 *)(src + (int64_t)z * slab_stride + (int64_t)tap * C + c);
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
#pragma unroll
        for (int d = 1; d < R; d <<= 1) {
            s.x += __shfl_xor(s.x, d); s.y += __shfl_xor(s.y, d); s.z += __shfl_xor(s.z, d); s.w += __shfl_xor(s.w, d);
        }
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
    const dim3 grid((unsigned)O, (unsigned)((C + 63) / 64));
    if (slabs >= 12)
        hipLaunchKernelGGL(finish_conv_kernel<8>, grid, dim3(1024), 0, st, part, slabs, O * (int64_t)taps * C, (uint16_t *)dW, C, taps, alpha);
    else
        hipLaunchKernelGGL(finish_conv_kernel<1>, grid, dim3(256), 0, st, part, slabs, O * (int64_t)taps * C, (uint16_t *)dW, C, taps, alpha);
    return hipGetLastError();
}

}  // namespace nm
