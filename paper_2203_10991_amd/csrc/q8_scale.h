// Device side of the 8-bit path's scales.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"          // LayerScale

namespace nm {

// The largest power-of-two scale of a maximum (bit pattern mb): s = 2^e with s * max <= top, e in [-126, 126]
__device__ __forceinline__ void scale_of_max(uint32_t mb, float top, float &s, float &inv)
{
    s = 1.0f; inv = 1.0f;
    if (mb != 0 && mb < 0x7f800000u && top > 0.0f && top < __builtin_inff()) {
        int em, et;
        const float fm = frexpf(__uint_as_float(mb), &em), ft = frexpf(top, &et);     // x = f * 2^e, f in [0.5, 1)
        int e = et - em - (ft >= fm ? 0 : 1);                                          // largest e with 2^e * max <= top
        e = e > 126 ? 126 : e < -126 ? -126 : e;
        s = __uint_as_float((uint32_t)(127 + e) << 23);
        inv = __uint_as_float((uint32_t)(127 - e) << 23);
    }
}

// A tensor's scale from the maxima that the workgroups of the pass over it left, found by every wave for itself: one 16-byte load, which belongs
// before the kernel's first loads, and a reduction over the lanes, which belongs behind them (in front of them it cost the cast and the prunes
// 2 us each).  All lanes of the wave have to be at both; `put`: the caller's first workgroup, which leaves the record for the kernels
// behind it.
__device__ __forceinline__ uint4 layer_peaks(const LayerScale &ls) { return ((const uint4 *)ls.peaks)[threadIdx.x & 63]; }     // (LAYER_PEAKS words, n of them written)
__device__ __forceinline__ float layer_scale(const LayerScale &ls, const uint4 &v, bool put)
{
    const int lane = threadIdx.x & 63;
    uint32_t m = 4 * lane < ls.n ? v.x : 0u;
    m = max(m, 4 * lane + 1 < ls.n ? v.y : 0u);
    m = max(m, 4 * lane + 2 < ls.n ? v.z : 0u);
    m = max(m, 4 * lane + 3 < ls.n ? v.w : 0u);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    float s, inv;
    scale_of_max(m, ls.top, s, inv);
    if (put && threadIdx.x == 0) *(float4 *)ls.rec = make_float4(s, inv, __uint_as_float(m), 0.0f);
    return s;
}

}  // namespace nm
