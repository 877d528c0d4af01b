// mac_xd.h -- what the kernels that multiply and accumulate without an x transform share (mac_xd.hip, mac_quads.hip).
#pragma once
#include "mac_common.h"
#include "split.h"

namespace znni {

struct XdArgs {
    FastDiv d_sub, d_pg, d_spr, d_nwg, d_Ny;
    const float2* X2;
    const half8* A;             // [pencil][slot][row tile][hi, lo][16 output images], 4 complex images each
    const float* rinv;          // [Mp] inverse of the power of two the kernel transforms of an output image carry, and two bits
    // what the kernel transforms are made of (k_kprep_xd): after the z stage, scales, twiddles along y
    const float2* A1;
    const float *row, *cinv;
    const float2* tw;
    float scale;
    int ky, fp;
    float2* Yd;
    unsigned ximg, yimg;        // elements between the rows of consecutive images in X2 / Yd
    size_t xpen, ypen;          // elements between the rows of pencils (oz, oy) and (oz + 1, oy)
    int xrow, yrow;             // ... of pencils (oz, oy) and (oz, oy + 1)
    int xblk, yblk;             // ... of four neighbouring x (xo) and the next four
    int f, fo, Mp, K, nx, nox, Ny;
    int nstrips, npencils, accumulate;
    int zc, Nz;                 // tiles: rows oz of stored kernel transforms, and of spectra
};

constexpr int XD_MAX_K = 9;     // taps along x at most: the halo of a staged row

// Slot of a pencil's stored kernel transforms -> image quad and tap: the order the contraction walks them in, chunks of four
// quads, inside a chunk tap by tap, quads fastest.
__device__ __forceinline__ void xd_slot(int slot, int K, int fq, int& quad, int& a)
{
    const int c = slot / (4 * K), s = slot - c * 4 * K, QC = min(4, fq - 4 * c);
    a = s / QC;
    quad = 4 * c + s - a * QC;
}

// The factor of the two unnormalised transforms, no power of two.
inline float xd_scale(const Dims& d) { return (float)(1.0 / ((double)d.Ny * d.Nz)); }

// mac_quads.hip: rows in blocks of four x, four neighbouring pencils a workgroup.  quads_strip: column tiles of a wave's strip.
znni_status launch_mac_quads(const LayerPlan& L, const XdArgs& g, hipStream_t st);
int quads_strip(const LayerPlan& L);

}  // namespace znni
