// The selection rules of the prune kernels, one block (pair or quad) at a time, and the small device helpers around them:
// streaming loads and stores, the stochastic rounding to e5m2.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "prune_common.h"

namespace nm {

// ------------------------------------------------------------------------------------
// MVUE 1:2 on one pair: returns kept position (0/1) and the kept value (unrounded).
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void select_1of2(float x0, float x1, uint32_t word, uint32_t &kept, float &value)
{
    const float m0 = fabsf(x0), m1 = fabsf(x1);
    const float s = m0 + m1;
    const float t = word_to_eps(word) * s;
    const bool keep0 = (m1 == 0.0f) | (t < m0);       // a zero never wins against a non-zero
    kept = keep0 ? 0u : 1u;
    value = copysignf(s, keep0 ? x0 : x1);
}

// ------------------------------------------------------------------------------------
// optimal MVUE 2:4 on one quad.
// Ranking key, most significant first: magnitude bits, then 3 - position (among equal
// magnitudes the higher position ranks lower), ..., the position itself, the sign.  The last two
// never decide an order (the code above them is unique); they ride along so that the kept
// elements' positions and signs come out of the sorted keys.  bf16 magnitudes leave the low
// 16 bits free, so the key fits 32 bits and is made straight from the packed row word (two
// columns per word): one merge of the column's half with the position constant, one rotate
// that moves the sign from the top to bit 0.  fp32 uses a 64-bit key.
// ------------------------------------------------------------------------------------
template <int DT> struct Key;
template <> struct Key<NM_DT_BF16> {
    typedef uint32_t type;
    // w: row word holding columns (2j, 2j+1); half: which of the two
    static __device__ __forceinline__ type make(const uint4 &v, int c, int pos)
    {
        const uint32_t w = (c >> 1) == 0 ? v.x : (c >> 1) == 1 ? v.y : (c >> 1) == 2 ? v.z : v.w;
        const uint32_t code = ((3u - (uint32_t)pos) << 14) | (uint32_t)pos;          // lands in key bits [16:15] and [2:1]
        const uint32_t d = (c & 1) ? ((w & 0xffff0000u) | code) : ((w << 16) | code);
        return __builtin_rotateleft32(d, 1);              // magnitude [31:17], 3-pos [16:15], pos [2:1], sign [0]
    }
    static __device__ __forceinline__ float mag(type k) { return __uint_as_float((k >> 1) & 0x7fff0000u); }
    static __device__ __forceinline__ uint32_t pos(type k) { return (k >> 1) & 3u; }
    static __device__ __forceinline__ float with_sign(float m, type k) { return __uint_as_float(__float_as_uint(m) | (k << 31)); }
};
template <> struct Key<NM_DT_F32> {
    typedef uint64_t type;
    static __device__ __forceinline__ type make(const uint4 &v, int c, int pos)
    {
        const uint32_t b = c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w;
        return ((uint64_t)(b & 0x7fffffffu) << 8) | ((3u - (uint32_t)pos) << 3) | ((uint32_t)pos << 1) | (b >> 31);
    }
    static __device__ __forceinline__ float mag(type k) { return __uint_as_float((uint32_t)(k >> 8)); }
    static __device__ __forceinline__ uint32_t pos(type k) { return ((uint32_t)k >> 1) & 3u; }
    static __device__ __forceinline__ float with_sign(float m, type k) { return __uint_as_float(__float_as_uint(m) | ((uint32_t)k << 31)); }
};

template <typename K> __device__ __forceinline__ void order2(K &a, K &b)
{
    const K lo = a < b ? a : b;
    const K hi = a < b ? b : a;
    a = lo;
    b = hi;
}
// ascending sort of four distinct keys.  64-bit keys: the 5-comparator network.  32-bit keys: the two middle keys
// come from three-input instructions -- with x <= X and y <= Y the sorted pairs and m = min(X, Y) >= min(x, y), the
// second key is the median and the third the maximum of {x, y, m} -- nine operations instead of ten.
__device__ __forceinline__ void sort4(uint64_t &k1, uint64_t &k2, uint64_t &k3, uint64_t &k4)
{
    order2(k1, k2); order2(k3, k4); order2(k1, k3); order2(k2, k4); order2(k2, k3);
}
__device__ __forceinline__ void sort4(uint32_t &k1, uint32_t &k2, uint32_t &k3, uint32_t &k4)
{
    order2(k1, k2); order2(k3, k4);
    const uint32_t x = k1, X = k2, y = k3, Y = k4;
    const uint32_t m = X < Y ? X : Y;
    k1 = x < y ? x : y;
    k4 = X < Y ? Y : X;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(k2) : "v"(x), "v"(y), "v"(m));
    asm("v_max3_u32 %0, %1, %2, %3" : "=v"(k3) : "v"(x), "v"(y), "v"(m));
}

// out0/out1: kept values in ascending position; nib = pos0 | pos1 << 2.  Straight-line code: the case
// analysis and the walk over the pair probabilities are lane masks and selects, no divergent branch.
template <int DT>
__device__ __forceinline__ void select_2of4(typename Key<DT>::type k1, typename Key<DT>::type k2, typename Key<DT>::type k3,
                                            typename Key<DT>::type k4, uint32_t word, float &out0, float &out1, uint32_t &nib)
{
    typedef Key<DT> KT;
    sort4(k1, k2, k3, k4);
    const float a1 = KT::mag(k1), a2 = KT::mag(k2), a3 = KT::mag(k3), a4 = KT::mag(k4);

    const float s12 = a1 + a2;
    const float s123 = s12 + a3;
    const float s = s123 + a4;
    const float u = fmaf(2.0f, a1, a3);                    // 2*a1 is exact: one rounding, as in (2*a1) + a3
    const bool case1 = a4 <= u;
    const bool case12 = case1 | (a4 <= s123);              // else case 3: a4 dominates

    // cumulative thresholds on t = eps * D.  Cases 1-2: D = 2(a1+a2+a3+a4), walk p13,p14,p23,p24,p34.
    // Case 3: D = a1+a2+a3, partner of a4 is a1 / a2 / a3; expressed in the same chain.
    const float t = word_to_eps(word) * (case12 ? s + s : s123);
    const float c13 = u - a4;                                                   // counts in case 1 only
    const float f4 = case12 ? 4.0f : 1.0f;                                     // (one select for both scaled thresholds: the products are exact)
    const float c14 = f4 * a1;
    const float d34 = s123 - a4;
    const float n23 = case1 ? (fmaf(2.0f, a2, a3) - a4) : (d34 + d34);
    const float c23 = 4.0f * a1 + n23;                                          // counts in cases 1-2 only
    const float c24 = f4 * s12;

    // the first threshold above t decides the pair: 13, 14, 23, 24, else 34 (case 3: 14, 24, else 34)
    const bool lt13 = case1 & (t < c13), lt14 = t < c14, lt23 = case12 & (t < c23), lt24 = t < c24;
    const bool first_is_1 = lt13 | lt14;
    const bool first_is_2 = lt23 | lt24;
    const bool second_is_3 = case12 & (lt13 | (!lt14 & lt23));
    const typename KT::type ka = first_is_1 ? k1 : (first_is_2 ? k2 : k3);
    const typename KT::type kb = second_is_3 ? k3 : k4;

    const float half_s = 0.5f * s;
    const float va = KT::with_sign(case12 ? half_s : s123, ka);                // a_i / p_i
    const float vb = KT::with_sign(case12 ? half_s : a4, kb);
    const uint32_t pa = KT::pos(ka), pb = KT::pos(kb);
    const bool swap = pa > pb;
    out0 = swap ? vb : va;
    out1 = swap ? va : vb;
    nib = swap ? (pb | (pa << 2)) : (pa | (pb << 2));
}

// ------------------------------------------------------------------------------------
// approx-MVUE 2:4 on one quad (Sec. 4.4): one element drawn with probability a_i/sum, a second from
// the other three with probability a_j/(sum - a_i); both kept with value a_k/p_k, p_k the section's
// inclusion probability, i.e.  sum / (1 + sum_{l != k} a_l/(sum - a_l)).  No ranking: position order.
// A draw is a threshold walk over the running sums (t = eps * total, first position whose running
// sum exceeds t); when none does -- rounding, or nothing non-zero left -- it falls on the last
// position with a non-zero magnitude, else on the lowest position not taken, so a zero never beats a
// non-zero and padding falls on the lowest-index zeros.  "sum - a_l" and the sum over l != k are
// formed from the other terms (no cancellation when one element carries the sum).  The six
// divisions are IEEE binary32 divisions.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void select_2of4_approx(float x0, float x1, float x2, float x3, uint32_t word1, uint32_t word2,
                                                   float &out0, float &out1, uint32_t &nib)
{
    // Straight-line code: draws are lane masks (one per position), everything else selects.
    const float m0 = fabsf(x0), m1 = fabsf(x1), m2 = fabsf(x2), m3 = fabsf(x3);
    const float c1 = m0 + m1, c2 = c1 + m2, total = c2 + m3;
    // first draw.  (t < total would pick position 3, and so does the fallback whenever m3 > 0; with m3 == 0 the
    // total equals c2 and the test cannot hold: one expression covers both.)
    const float t = word_to_eps(word1) * total;
    const bool w0 = t < m0, w1 = t < c1, w2 = t < c2;                           // walk
    const bool n0 = m0 > 0.0f, n1 = m1 > 0.0f, n2 = m2 > 0.0f, n3 = m3 > 0.0f;
    const bool i0 = w0 | (!w1 & !w2 & !n3 & !n2 & !n1);                         // (fallback on position 0: nothing non-zero above it)
    const bool i1 = !w0 & (w1 | (!w2 & !n3 & !n2 & n1));
    const bool i2 = !w0 & !w1 & (w2 | (!n3 & n2));
    const bool i3 = !w0 & !w1 & !w2 & n3;
    // second draw on the block without the first element
    const float r0 = i0 ? 0.0f : m0, r1 = i1 ? 0.0f : m1, r2 = i2 ? 0.0f : m2, r3 = i3 ? 0.0f : m3;
    const float d1 = r0 + r1, d2 = d1 + r2, rest = d2 + r3;
    const float t2 = word_to_eps(word2) * rest;
    const bool u0 = t2 < r0, u1 = t2 < d1, u2 = t2 < d2;
    const bool q0 = r0 > 0.0f, q1 = r1 > 0.0f, q2 = r2 > 0.0f, q3 = r3 > 0.0f;
    const bool none = !q0 & !q1 & !q2 & !q3;                                    // nothing non-zero left: lowest position not taken
    const bool fall = !u0 & !u1 & !u2;
    const bool j0 = u0 | (fall & ((!q3 & !q2 & !q1 & q0) | (none & !i0)));
    const bool j1 = !u0 & (u1 | (!u2 & ((!q3 & !q2 & q1) | (none & i0))));
    const bool j2 = !u0 & !u1 & (u2 | (!q3 & q2));
    const bool j3 = fall & q3;
    // kept values: sum / (1 + sum over the other three of a_l / (sum - a_l)), "sum - a_l" from the other three
    const float s23 = m2 + m3;
    const float o0 = m1 + s23, o1 = m0 + s23, o2 = c1 + m3, o3 = c2;
    const float e0 = m0 / o0, e1 = m1 / o1, e2 = m2 / o2, e3 = m3 / o3;         // (0/0 of a zero element is discarded below)
    const float v0 = n0 ? e0 : 0.0f, v1 = n1 ? e1 : 0.0f, v2 = n2 ? e2 : 0.0f, v3 = n3 ? e3 : 0.0f;
    const float di = 1.0f + ((((i0 ? 0.0f : v0) + (i1 ? 0.0f : v1)) + (i2 ? 0.0f : v2)) + (i3 ? 0.0f : v3));
    const float dj = 1.0f + ((((j0 ? 0.0f : v0) + (j1 ? 0.0f : v1)) + (j2 ? 0.0f : v2)) + (j3 ? 0.0f : v3));
    const float xi = i0 ? x0 : i1 ? x1 : i2 ? x2 : x3;
    const float xj = j0 ? x0 : j1 ? x1 : j2 ? x2 : x3;
    const float vi = copysignf(total / di, xi), vj = copysignf(total / dj, xj);
    const uint32_t pi = i0 ? 0u : i1 ? 1u : i2 ? 2u : 3u, pj = j0 ? 0u : j1 ? 1u : j2 ? 2u : 3u;
    const bool swap = pi > pj;
    out0 = swap ? vj : vi;
    out1 = swap ? vi : vj;
    nib = swap ? (pj | (pi << 2)) : (pi | (pj << 2));
}

// ------------------------------------------------------------------------------------
// MVUE 1:4 on one quad (appendix, additional sparsity results: MVUE 1:2 on a block of four): position k is kept
// with probability a_k/sum and emits sign(x_k) * sum.  Same threshold walk and fallback as the draws above.
// Stored in the 2:4 container: the quad's other slot is a +0 at the lowest other position.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void select_1of4(float x0, float x1, float x2, float x3, uint32_t word,
                                            float &out0, float &out1, uint32_t &nib)
{
    const float m0 = fabsf(x0), m1 = fabsf(x1), m2 = fabsf(x2), m3 = fabsf(x3);
    const float c1 = m0 + m1, c2 = c1 + m2, total = c2 + m3;
    const float t = word_to_eps(word) * total;
    const bool w0 = t < m0, w1 = t < c1, w2 = t < c2;
    const bool n1 = m1 > 0.0f, n2 = m2 > 0.0f, n3 = m3 > 0.0f;
    const bool i0 = w0 | (!w1 & !w2 & !n3 & !n2 & !n1);
    const bool i1 = !w0 & (w1 | (!w2 & !n3 & !n2 & n1));
    const bool i2 = !w0 & !w1 & (w2 | (!n3 & n2));
    const float xi = i0 ? x0 : i1 ? x1 : i2 ? x2 : x3;
    const float v = copysignf(total, xi);
    const uint32_t k = i0 ? 0u : i1 ? 1u : i2 ? 2u : 3u;
    out0 = i0 ? v : 0.0f;
    out1 = i0 ? 0.0f : v;
    nib = i0 ? 4u : (k << 2);                  // (0, 1) when position 0 is kept, else (0, k)
}

// ------------------------------------------------------------------------------------
// Greedy N:M (the comparison method of the paper's tables, Sec. 4.1 ablation and Sec. 5: keep the n largest
// magnitudes of the block, values unchanged).  Deterministic: no random words.  Among equal magnitudes the lower
// position is kept -- the order of the ranking keys above.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void select_greedy_1of2(float x0, float x1, uint32_t &kept, float &value)
{
    const bool keep1 = fabsf(x1) > fabsf(x0);
    kept = keep1 ? 1u : 0u;
    value = keep1 ? x1 : x0;
}
template <int DT>
__device__ __forceinline__ void select_greedy_2of4(typename Key<DT>::type k1, typename Key<DT>::type k2, typename Key<DT>::type k3,
                                                   typename Key<DT>::type k4, float &out0, float &out1, uint32_t &nib)
{
    typedef Key<DT> KT;
    sort4(k1, k2, k3, k4);
    const float va = KT::with_sign(KT::mag(k3), k3), vb = KT::with_sign(KT::mag(k4), k4);
    const uint32_t pa = KT::pos(k3), pb = KT::pos(k4);
    const bool swap = pa > pb;
    out0 = swap ? vb : va;
    out1 = swap ? va : vb;
    nib = swap ? (pb | (pa << 2)) : (pa | (pb << 2));
}

// ------------------------------------------------------------------------------------
// Streaming (non-temporal) forms of a 16-byte load and store
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
// (the pointers are to global memory; said explicitly, because an address that went through an opaque asm statement
// would otherwise be loaded from with the generic form, which counts as an LDS operation too)
#define NM_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ uint4 load_stream(const void *p)
{
    const u32x4_t t = __builtin_nontemporal_load((const NM_GLOBAL u32x4_t *)p);
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint4 load_global(const void *p)
{
    const u32x4_t t = *(const NM_GLOBAL u32x4_t *)p;
    return make_uint4(t.x, t.y, t.z, t.w);
}
// 8-byte pieces (the other half of the vector is zero and never read)
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 load_stream8(const void *p)
{
    const u32x2_t t = __builtin_nontemporal_load((const NM_GLOBAL u32x2_t *)p);
    return make_uint4(t.x, t.y, 0u, 0u);
}
__device__ __forceinline__ uint4 load_global8(const void *p)
{
    const u32x2_t t = *(const NM_GLOBAL u32x2_t *)p;
    return make_uint4(t.x, t.y, 0u, 0u);
}
// the same pieces through a buffer descriptor: zeros past its bound, nothing stored past it
template <int BYTES> __device__ __forceinline__ uint4 buffer_piece(__amdgpu_buffer_rsrc_t r, uint32_t offset)
{
    if constexpr (BYTES == 16) {
        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(r, (int)offset, 0, 0);
        return make_uint4(t.x, t.y, t.z, t.w);
    } else {
        const u32x2_t t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)offset, 0, 0);
        return make_uint4(t.x, t.y, 0u, 0u);
    }
}
// NT: the streaming form
template <int BYTES, bool NT = false> __device__ __forceinline__ void buffer_put_piece(__amdgpu_buffer_rsrc_t r, uint32_t offset, const uint4 &v)
{
    if constexpr (BYTES == 16) { const u32x4_t t = {v.x, v.y, v.z, v.w}; __builtin_amdgcn_raw_buffer_store_b128(t, r, (int)offset, 0, NT ? 2 : 0); }
    else { const u32x2_t t = {v.x, v.y}; __builtin_amdgcn_raw_buffer_store_b64(t, r, (int)offset, 0, NT ? 2 : 0); }
}
__device__ __forceinline__ void store_stream(void *p, const uint4 &v)
{
    const u32x4_t t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, (u32x4_t *)p);
}

// ------------------------------------------------------------------------------------
// Stochastic rounding to e5m2 with 16 random bits: with lo <= |x| < hi neighbours on the e5m2 grid and
// f = (|x| - lo)/(hi - lo), the result is hi iff r16 + floor(f * 2^16) >= 2^16.
// The rounding itself is one instruction: v_cvt_sr_bf8_f32 adds the top 21 bits of its random operand to the 21
// mantissa bits it discards (subnormal results: to the bits below the 2^-16 step) and truncates, which with the 16
// rounding bits in the operand's top half and zeros below them is exactly the rule above -- checked against the
// integer formulation for every rounding word over a million inputs of every exponent.  It overflows to infinity
// where this format saturates, so the value is clamped to +-57344 first; the code lands in byte BYTE of `word`.
template <int BYTE>
__device__ __forceinline__ uint32_t sr_e5m2_into(uint32_t word, float x, uint32_t r_top)
{
    const float c = __builtin_amdgcn_fmed3f(x, -57344.0f, 57344.0f);
    return (uint32_t)__builtin_amdgcn_cvt_sr_bf8_f32(c, (int)r_top, (int)word, BYTE);
}

}  // namespace nm
