// kprep.h -- the kernel transform's first stage and its scales: what mac.hip and passes_fused.hip share.
#pragma once
#include "znni_internal.h"

namespace znni {

constexpr int KPREP_OZ = 16;        // consecutive oz of a thread (k_kprep_z)

// Scales of the kernel transforms (kprep_row_scale in mac.hip says what they are).  Sums of kernels' magnitudes of an output image
// more than 2^UNEVEN apart are uneven.
constexpr int UNEVEN = 14;
// Exponent of the power of two that an input image's values are scaled by.
__device__ __forceinline__ int kprep_col_exp(float cmax, float most)
{
    const int t = (int)(__float_as_uint(cmax) >> 23) - (int)(__float_as_uint(most) >> 23);
    return cmax == 0.f || t >= -8 ? 0 : (t >= -24 ? t / 2 : max(t + 12, -60));
}
// The power of two of output image j and its inverse, from the largest, the smallest and (less one) the smallest sum that is not
// zero of its kernels' magnitudes.
__device__ __forceinline__ void kprep_row_store(const SplitScales& S, int j, float m, unsigned lo, unsigned lo1)
{
    const bool small = (int)lo1 < (int)__float_as_uint(m) - (UNEVEN << 23) && lo1 != ~0u;
    const unsigned bits = (small || lo == 0 ? 0x80000000u : 0u) | (small ? 1u : 0u);
    const int e = max(min(14 - ((int)((__float_as_uint(m) >> 23) & 255u) - 127), 120), -120);
    S.row[j] = m > 0.f ? __uint_as_float((unsigned)(127 + e) << 23) : 1.f;
    S.rinv[j] = m > 0.f ? __uint_as_float((unsigned)(127 - e) << 23 | bits) : 1.f;
}

}  // namespace znni
