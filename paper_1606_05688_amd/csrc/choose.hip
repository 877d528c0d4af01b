// choose.hip -- which primitive to run a convolutional layer with (host only), and the call that does so.
//
// Section VII: every layer can be computed by several primitives and the fastest one is picked per layer; the
// paper measures each candidate (Table IV lists the winners) and prunes the search with a kernel-size rule.
// Here the pick comes from a two-term cost model per primitive, with rates measured on one MI355X:
//
//   transform route:  bytes moved by the transform passes of the route that the planner takes and by the kernel
//                     preparation over the HBM rate those kernels reach (lower for transform lengths served by the
//                     generic pass kernel), plus the multiply-accumulate's matrix-core work or, where x is not
//                     transformed, the spectra it moves if they take longer, plus a fixed cost for every launch;
//   direct route:     the estimate of the kernel that would run (direct.hip, direct_split.hip, direct_first.hip): its walks over
//                     tiles, taps and staged values, and the tensors it moves.
//
// The model only has to rank the two; it is not used for anything else.  Over 23318 random layers that both take, the pick by these
// estimates is 0.5 % slower than the faster one on average, 685 by more than 5 %.  Where direct sums are the closer ones to 64 bits, the
// transform has to be ahead by bare rates as well (direct_stands): 1.0 % and 1083 with that.
#include "direct_split.h"
#include "mac_common.h"

namespace znni {

// measured rates (MI355X)
constexpr double kPassBytesPerSecFast = 5.3e12;     // in-register pass kernels
constexpr double kPassBytesPerSecGeneric = 2.0e12;  // generic LDS pass kernels
constexpr double kPrepBytesPerSec = 4.5e12;         // kernel preparation (write-bound)
constexpr double kMacFlopsPerSec = 110e12;          // issued matrix-core flops of the multiply-accumulate (S = 1 form)
constexpr double kLaunchSec = 3.5e-6;

// The route and its passes as the planner has them: bytes of every stage of the call that would run.
double route_seconds(const LayerPlan& L)
{
    if (L.tiles) return tiles_seconds(L);
    double hb[ZNNI_NUM_STAGES], fl[ZNNI_NUM_STAGES];
    plan_work(L, 0, hb, fl);
    const Dims& d = L.d;
    const int S = L.S;
    const double bins = (double)d.zc * d.Ny, bank = 8.0 * bins * d.kx * L.fp * L.Mp;
    double t = bank / kPrepBytesPerSec;
    int launches = 3;                                        // kernels (behind the tables), multiply-accumulate
    const int len[ZNNI_NUM_STAGES] = {0, d.Nz, d.Ny, d.Nx, 0, d.Nx, d.Ny, d.Nz};
    for (int q = 0; q < ZNNI_NUM_STAGES; ++q)
        if (len[q] && hb[q] > 0) {
            t += hb[q] / (fast_pass_available(len[q]) ? kPassBytesPerSecFast : kPassBytesPerSecGeneric);
            ++launches;
        }
    if (L.xdirect) {
        // bound by its split products or by the spectra it reads and writes
        const double by = 8.0 * bins * ((double)L.nimg * d.nx + (double)L.nimgo * d.nox) + bank;
        const double ops = 24.0 * d.kx * L.fp * (double)L.Mp * S * d.nox * bins;
        t += by / kPassBytesPerSecFast > ops / MAC_SPLIT_FLOPS ? by / kPassBytesPerSecFast : ops / MAC_SPLIT_FLOPS;
    } else if (mac_batch_preferred(L)) {
        t += MAC_BATCH_SEC_PER_VALUE * L.fp * (double)L.Mp * d.Nx * bins * ((S + 15) / 16);
    } else {
        // three real matrix products per complex one, contraction over (input image, x tap), every column
        t += 6.0 * d.kx * L.fp * (double)L.Mp * S * d.Nx * bins / kMacFlopsPerSec;
    }
    return t + launches * kLaunchSec;
}

static double fft_seconds(int S, int f, int fo, const int n[3], const int k[3])
{
    LayerPlan L;
    if (make_plan(S, f, fo, n, k, 0, nullptr, &L)) return -1.0;
    // (the estimate of tiles is that of a call; that of whole planes, which serves to rank routes, is low by 20 to 35 %)
    return L.tiles ? route_seconds(L) : 1.25 * route_seconds(L);
}

// Whether a layer stays with direct sums though transforms are estimated to be the faster.  Direct sums of K products are 1.8e-8 sqrt(K)
// of the result off its 64-bit value (1.4e-8 on split halves), transforms 1.9e-7 to 2.2e-7 whatever K (108 layers that the two
// estimates disagree on): sums of up to 110 products come out closer directly, by 1.2 times on average up to 100 and 1.8 at 40 (on split
// halves up to 190); at 114 to 136 the two are level.  So those leave the direct kernels only where whole planes would be faster by
// rates alone: 621 of 23318 random layers stay, 1.19 times as long as by transforms on average, 2.6 at most.
static bool direct_stands(int S, int f, int fo, const int n[3], const int k[3])
{
    constexpr double kDirectFlops = 80e12, kDirectFlopsFew = 60e12;      // windows of 27 taps and more, of fewer
    constexpr double kDirectWrite = 3.6e12, kSplitBytes = 2.6e12, kSplitFlops = 75e12;
    LayerPlan L;
    SplitPlan P;
    const int taps = k[0] * k[1] * k[2];
    if ((long long)f * taps > 190 || make_whole_plan(S, f, fo, n, k, 0, nullptr, &L)) return false;
    const bool split = split_plan(S, f, fo, L.d, &P);
    if (!split && f * taps > 110) return false;
    const double ovox = (double)L.d.nox * L.d.noy * L.d.noz, wr = 4.0 * S * fo * ovox;
    double t;
    if (split) {
        const double by = (wr + 4.0 * S * f * n[0] * n[1] * n[2]) / kSplitBytes;
        const double fl = 2.0 * S * 32 * P.nsteps * 16.0 * P.RT * P.nmblk * ovox / kSplitFlops;
        t = by > fl ? by : fl;
    } else {
        // products and writing, or a workgroup's walk over its steps of four taps: matrix instructions of 32 cycles and 450 of latency
        const double taps4 = (taps + 3) / 4 * 4, Mp = (fo + 15) / 16 * 16, rows = Mp / 16 < 5 ? Mp / 16 : 5;
        const double walk = f * taps4 / 4 * (rows * 4 * 32 + 450) / 2.2e9;
        t = 2.0 * S * f * taps4 * Mp * ovox / (taps >= 27 ? kDirectFlops : kDirectFlopsFew) + wr / kDirectWrite;
        if (t < walk) t = walk;
    }
    return t + 2 * kLaunchSec < route_seconds(L);
}

}  // namespace znni

using namespace znni;

extern "C" {

znni_status znni_conv3d_choose_v(int S, int f, int fo, const int n[3], const int k[3], int* primitive,
                                 float est_ms[2])
{
    if (!primitive) return ZNNI_ERR_NULL;
    size_t bf = 0, bd = 0;
    const znni_status rf = znni_conv3d_fft_workspace_v(S, f, fo, n, k, &bf);
    const znni_status rd = znni_conv3d_direct_workspace_v(S, f, fo, n, k, &bd);
    if (rf != ZNNI_OK && rd != ZNNI_OK) return rf;          // bad shape, or neither primitive takes it
    const double tf = rf == ZNNI_OK ? fft_seconds(S, f, fo, n, k) : -1.0;
    const double td = rd == ZNNI_OK ? direct_seconds(S, f, fo, n, k) : -1.0;
    if (est_ms) { est_ms[ZNNI_PRIMITIVE_FFT] = (float)(tf * 1e3); est_ms[ZNNI_PRIMITIVE_DIRECT] = (float)(td * 1e3); }
    if (tf < 0) *primitive = ZNNI_PRIMITIVE_DIRECT;
    else if (td < 0) *primitive = ZNNI_PRIMITIVE_FFT;
    else *primitive = td < tf || direct_stands(S, f, fo, n, k) ? ZNNI_PRIMITIVE_DIRECT : ZNNI_PRIMITIVE_FFT;
    return ZNNI_OK;
}

znni_status znni_conv3d_workspace_v(int S, int f, int fo, const int n[3], const int k[3], size_t* bytes)
{
    if (!bytes) return ZNNI_ERR_NULL;
    int prim = 0;
    znni_status rc = znni_conv3d_choose_v(S, f, fo, n, k, &prim, nullptr);
    if (rc) return rc;
    return prim == ZNNI_PRIMITIVE_DIRECT ? znni_conv3d_direct_workspace_v(S, f, fo, n, k, bytes)
                                         : znni_conv3d_fft_workspace_v(S, f, fo, n, k, bytes);
}

znni_status znni_conv3d_v(int S, int f, int fo, const int n[3], const int k[3], const float* in, const float* w,
                          const float* bias, float* out, unsigned flags, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    int prim = 0;
    znni_status rc = znni_conv3d_choose_v(S, f, fo, n, k, &prim, nullptr);
    if (rc) return rc;
    if (prim == ZNNI_PRIMITIVE_DIRECT) {
        if (flags & ZNNI_MAC_REFERENCE) return ZNNI_ERR_FLAGS;
        // the transform route's stricter alignment is asked of both, so a call does not depend on the pick
        if (in && w && out && (((uintptr_t)in | (uintptr_t)w | (uintptr_t)out) & 15u)) return ZNNI_ERR_ALIGN;
        // the hints that pick a multiply-accumulate form mean nothing to the direct route: validated, then dropped
        // (at most one, as on the transform route); the direct route stores no kernel transforms a later call
        // could reuse, so ZNNI_KEEP_KERNELS is dropped as well: the bank is rearranged again, which is always right; it
        // has no transform passes either
        const unsigned forms = flags & (unsigned)(ZNNI_MAC_SINGLE | ZNNI_MAC_BATCH | ZNNI_MAC_XDIRECT | ZNNI_MAC_XBLOCK);
        if (forms & (forms - 1)) return ZNNI_ERR_FLAGS;
        return znni_conv3d_direct_v(S, f, fo, n, k, in, w, bias, out,
                                    flags & ~(forms | (unsigned)(ZNNI_KEEP_KERNELS | ZNNI_PASSES_REFERENCE)), workspace,
                                    workspace_bytes, stream);
    }
    return znni_conv3d_fft_v(S, f, fo, n, k, in, w, bias, out, flags, workspace, workspace_bytes, stream);
}

}  // extern "C"
