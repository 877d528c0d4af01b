// direct_split.h -- plan and launcher of the split-half direct convolution (direct_split.hip).
#pragma once
#include "znni_internal.h"

namespace znni {

constexpr int SPLIT_NT = 256;     // threads per workgroup
constexpr int SPLIT_UNITS = 4;    // staged (image octet, position) units per thread, at most

struct SplitPlan {
    int RT, CT, nmblk, noct, nslots, nsteps;
    int TX, TY, TZ16, nz, npos, ntiles;
    size_t lds, bytes;            // bytes: kernel bank and row scales
};

// Whether (and how) a layer runs on this kernel; d needs image, kernel and output sizes only.
bool split_plan(int S, int f, int fo, const Dims& d, SplitPlan* P);
znni_status launch_direct_split(const SplitPlan& P, int S, int f, int fo, const Dims& d, const float* in, const float* w,
                                const float* bias, float* out, int relu, void* workspace, hipStream_t st);

}  // namespace znni
