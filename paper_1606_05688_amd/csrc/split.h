// split.h -- fp32 values on the fp16 matrix instructions: two halves per value and power-of-two scales (see mac_xd.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace znni {

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

// Largest magnitude of a thread's values so far and two more: one instruction (fmaxf first quiets each operand).
__device__ __forceinline__ void max3_abs(float& m, float a, float b)
{
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
}
// Largest value of a wave (non-negative floats, compared as integers: a NaN counts as the largest).
__device__ __forceinline__ unsigned wave_max(float m)
{
    unsigned v = __float_as_uint(m);
#define ZNNI_DPP(CTRL, ROWS) v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false))
    ZNNI_DPP(0x111, 0xf);        // row_shr 1, 2, 4, 8: lane 15 of every row of sixteen holds the row's largest
    ZNNI_DPP(0x112, 0xf);
    ZNNI_DPP(0x114, 0xf);
    ZNNI_DPP(0x118, 0xf);
    ZNNI_DPP(0x142, 0xa);        // row_bcast 15, 31: lane 63 holds the wave's
    ZNNI_DPP(0x143, 0xc);
#undef ZNNI_DPP
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

}  // namespace znni
