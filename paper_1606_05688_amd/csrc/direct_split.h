// direct_split.h -- plans and launchers of the direct convolutions on split halves (direct_split.hip, direct_first.hip).
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
double split_us(const SplitPlan& P, int S, int f, int fo, const Dims& d);     // its estimated time
znni_status launch_direct_split(const SplitPlan& P, int S, int f, int fo, const Dims& d, const float* in, const float* w,
                                const float* bias, float* out, int relu, void* workspace, hipStream_t st);

// Layers of few taps, whose result's writing is the bound (direct_first.hip).
struct FirstPlan {
    int RTW, nmblk;               // row tiles (16 output images) of a workgroup, blocks of them
    int TZ, TY, total, tiles;     // columns and rows of a tile, its staged values, tiles
    double us;                    // estimated time
};

// Whether (and how) this kernel takes a layer.
bool first_plan(int S, int f, int fo, const Dims& d, FirstPlan* P);
znni_status launch_direct_first(const FirstPlan& P, int f, int fo, const Dims& d, const float* in, const float* w, const float* bias,
                                float* out, int relu, hipStream_t st);

// Estimated time of a direct convolution, by the kernel that would compute it (negative where none does).
double direct_seconds(int S, int f, int fo, const int n[3], const int k[3]);

}  // namespace znni
