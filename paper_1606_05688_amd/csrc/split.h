// split.h -- fp32 values on the fp16 matrix instructions: two halves per value and power-of-two scales (see mac_xd.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace znni {

typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Division by a number known at launch: a high product, at most one too large, and a correction.
struct FastDiv {
    unsigned d, m;
    void set(unsigned n) { d = n; m = n > 1 ? (unsigned)((1ull << 32) / n) + 1u : 0u; }
    __device__ __forceinline__ unsigned div(unsigned n) const
    {
        if (d == 1) return n;
        const unsigned q = __umulhi(n, m);
        return q * d > n ? q - 1 : q;
    }
};

// The largest finite magnitude that decides a scale sits at 2^SPLIT_TOP.
constexpr int SPLIT_TOP = 14;
// Power-of-two exponent that brings values of magnitude m (finite) to 2^SPLIT_TOP; both it and its negative are exponents
// of normal numbers.
__device__ __forceinline__ int split_exp(float m)
{
    const int e = (int)((__float_as_uint(m) >> 23) & 255u) - 127;
    return min(SPLIT_TOP - e, 126);
}
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }

__device__ __forceinline__ void split2(float v, float s, _Float16& hi, _Float16& lo)
{
    hi = (_Float16)(v * s);
    lo = (_Float16)fmaf(v, s, -(float)hi);
}

// A value as three halves, the second and third 2^11 and 2^22 times what is left to them: exact where v * s lies between 2^-23 and
// 2^15 (a half's last place is 2^-24 at least, so the third's 2^-46).
constexpr float SPLIT3_STEP = 1.f / 2048;
__device__ __forceinline__ void split3(float v, float s, _Float16& hi, _Float16& mid, _Float16& lo)
{
    hi = (_Float16)(v * s);
    const float r = fmaf(v, s, -(float)hi) * 2048.f;
    mid = (_Float16)r;
    lo = (_Float16)((r - (float)mid) * 2048.f);
}

// (x, -y) as two pairs of halves, the same values as split2 gives: every half leaves one mixed-precision instruction where
// it belongs (a product, its conversion, the difference and the packing of pairs took three a value).
__device__ __forceinline__ void split_conj(float x, float y, float s, unsigned& hi, unsigned& lo)
{
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(hi) : "v"(x), "v"(s));
    asm("v_fma_mixhi_f16 %0, -%1, %2, 0" : "+v"(hi) : "v"(y), "v"(s));
    asm("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(lo) : "v"(x), "v"(s), "v"(hi));
    asm("v_fma_mixhi_f16 %0, -%1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(lo) : "v"(y), "v"(s), "v"(hi));
}

// A value of 2^-17 of the largest still has all its 22 bits; below that a bit goes with every power of two.  Where a value
// (that is not zero) lies more than 2^-SPLIT_SPAN below the largest of its group, the group is multiplied in fp32.
constexpr int SPLIT_SPAN = 19;

// Largest magnitude of a thread's values so far and two more: one instruction (fmaxf first quiets each operand; NaNs are
// passed over).
__device__ __forceinline__ void max3_abs(float& m, float a, float b)
{
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
}
// Largest (smallest) value of a wave, as unsigned integers (non-negative floats keep their order).
#define ZNNI_DPP(F, OLD, CTRL, ROWS) v = F(v, (unsigned)__builtin_amdgcn_update_dpp((int)(OLD), (int)v, CTRL, ROWS, 0xf, false))
// row_shr 1, 2, 4, 8: lane 15 of every row of sixteen holds the row's; row_bcast 15, 31: lane 63 holds the wave's
#define ZNNI_DPP_ALL(F, OLD)                                                                             \
    ZNNI_DPP(F, OLD, 0x111, 0xf); ZNNI_DPP(F, OLD, 0x112, 0xf); ZNNI_DPP(F, OLD, 0x114, 0xf);             \
    ZNNI_DPP(F, OLD, 0x118, 0xf); ZNNI_DPP(F, OLD, 0x142, 0xa); ZNNI_DPP(F, OLD, 0x143, 0xc)
__device__ __forceinline__ unsigned wave_max(float m)
{
    unsigned v = __float_as_uint(m);
    ZNNI_DPP_ALL(max, 0u);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned wave_min(unsigned v)
{
    ZNNI_DPP_ALL(min, ~0u);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
#undef ZNNI_DPP_ALL
#undef ZNNI_DPP

// A magnitude as an integer that orders like it, except that zero is the largest: twice the bits without the sign, less one.
__device__ __forceinline__ unsigned small_code(float v) { return (__float_as_uint(v) << 1) - 1u; }
// Whether the smallest such code of a group is out of the range that halves hold next to its largest magnitude (its bits).
__device__ __forceinline__ bool split_too_wide(unsigned largest, unsigned code, int span = SPLIT_SPAN)
{
    const int e = (int)(largest >> 23) - span;
    return e > 0 && code < ((unsigned)e << 24) - 1u;
}

}  // namespace znni
