// api.hip -- the exported C ABI: argument validation, workspace planning, and the stage sequence of the
// GPU algorithm of Section IV-B-2 (Algorithm 3): transform the images, multiply-accumulate per bin with the
// kernel transforms, inverse-transform the output images.  All validation happens before the first HIP call.
#include <stdint.h>

#include <mutex>

#include "mac_common.h"
#include "znni_internal.h"

// Scratch memory of znni_conv3d_fft_static_v, the entry point for callers that cannot allocate: one array per GPU,
// placed by the loader when the library's code is loaded on that GPU and held until the process ends.  In host
// code this name is only a handle for hipGetSymbolAddress; kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[ZNNI_STATIC_SCRATCH_BYTES];

namespace znni {

// Transform size for an image edge n: the smallest length >= n that the in-register pass kernels serve (46
// members of the 2^a 3^b 5^c 7^d family from 8 to 1024, never more than 20 % above n); below 7 the edge itself (all
// of 1..6 are members), transformed by the generic pass kernels.  A layer's cost grows in proportion to the length,
// and the generic kernels run at well under half the speed per element, so a nearer generic length never pays.
static int fft_size(int n)
{
    if (n < 1) return 0;
    if (n < 7) return n;
    for (int m = n; m <= ZNNI_MAX_FFT; ++m)
        if (fast_pass_available(m)) return m;
    return 0;
}

// Radix schedule: odd primes first, then the power of two as 8s with a 4,4 / 4 / 2 tail.
static void make_fft_plan(int N, FftPlan* P)
{
    P->N = N;
    P->nstages = 0;
    int m = N;
    for (int p : {7, 5, 3})
        while (m % p == 0) { P->radix[P->nstages++] = p; m /= p; }
    int a = 0;
    while (m > 1) { m >>= 1; ++a; }
    if (a == 1) { P->radix[P->nstages++] = 2; a = 0; }
    if (a % 3 == 1) { P->radix[P->nstages++] = 4; P->radix[P->nstages++] = 4; a -= 4; }
    if (a % 3 == 2) { P->radix[P->nstages++] = 4; a -= 2; }
    while (a > 0) { P->radix[P->nstages++] = 8; a -= 3; }
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Whether a layer that does not go four planes at a time (pick_planes) runs without transforming its x axis (mac_xd.hip).  A flag
// that names a multiply-accumulate form decides; otherwise that route is taken, provided the y transform has an in-register
// kernel (only those read the transposed layout), except for small images with many inputs or many images: with fused z+y
// kernels on both sides the fully transformed route has as many passes, and a kernel-spectrum value generated once per bin
// serves all inputs.  Measured, whole layer, untransformed against fully transformed: 80 -> 80 images of 100^3, 5^3 kernels
// 1.34 against 1.96 ms; 32 -> 32 of 64^3, 7^3 0.137 against 0.174; 8 x 32 -> 32 of 130^3, 5^3 (no fused kernels) 5.9 against 8.9;
// 32 x 20 -> 20 of 40 x 128 x 100, 3^3 2.92 against 4.06.  With fused kernels and more than 8 inputs: 16 x 80 -> 80 of 80^3, 5^3
// 7.5 against 7.0; with at most 8 inputs and k * S >= 32 it is ahead or level above length 64 (8 x 80 -> 80 of 99^3, 5^3 7.6
// against 10.1, 8 x 48 -> 48 of 72^3, 4^3 1.48 against 1.63, 8 x 16 -> 16 of 120^3, 5^3 2.04 against 2.01).
static bool pick_untransformed_x(const LayerPlan& L, unsigned flags)
{
    if (flags & (ZNNI_MAC_REFERENCE | ZNNI_MAC_SINGLE | ZNNI_MAC_BATCH)) return false;
    const bool batch = mac_batch_preferred(L);
    // (batches with rows of the output shorter than that leave most of a column tile idle; around the line the two are level: 15 x
    // 93 -> 44 of 27 x 21 x 30, 7 x 5 x 2 kernels 0.371 against 0.382 ms)
    if (!(fused_fwd_zy_available(L) && fused_inv_yz_available(L))) return !batch || L.d.nox >= 32;
    if (batch) return L.S <= 8 && L.d.Ny > 64;
    if (L.S >= 8) return false;
    // Above length 64 four passes without any along x are faster than two fused ones with two along x: over 245 random layers of
    // up to 7 inputs 0.5 % off the faster route on average.  Up to there the fused kernels gain with every image, the untransformed route with every product per image (its multiply-accumulate is the faster
    // one), and where there are few pencils for long sums nothing hides a workgroup's walk.  Over 204 random layers too large for
    // four planes this is 3.3 % off the faster route on average, never transforming x 2.8 %, always doing so 13.6 %.  (It is kept for
    // the many small layers below, where it says which route four planes stand against.)  Untransformed against transformed, us:
    // 10 -> 44 images of 59^3, 3^3 kernels 80 against 88; 18 -> 122 of 41^3, 6^3 138 against 177; 3 x 83 -> 6 of 41^3, 5^3 192 against
    // 230; 7 -> 1 of 65^3, 7^3 55 against 74; 7 x 88 -> 1 of 37^3, 2^3 250 against 197; 7 x 103 -> 7 of 54^3, 3^3 777 against 647.
    // The largest loss: 7 x 4 -> 65 of 37^3, 9 x 6 x 3 115 against 180.
    const int pencils = L.d.zc * L.d.Ny;
    if (L.d.Ny > 64) return true;
    if (L.S * L.f <= 80) return L.S * L.fo <= 300 && 2 * L.f * L.d.kx <= 3 * pencils;
    return pencils >= 512 && (long long)L.f * L.fo * L.d.kx >= 8ll * L.S * (L.f + L.fo);
}

// ... and whether it applies the kernel's taps along x through length-8 transforms of overlapping blocks
// (mac_xb.hip) rather than as shifted reads: only where the call asks for that form.  Measured, shifted reads on split
// halves against blocks on fp32, whole layer: 48 -> 48 images of 320^3, 5^3 kernels 17.0 against 17.2 ms; 48 -> 48 of 160^3,
// 5^3 2.21 against 2.53; 80 -> 80 of 200^3, 5^3 9.3 against 10.4; 80 -> 80 of 100^3, 5^3 1.6 against 1.7; and the closer
// results (mac_xd.hip).
static bool pick_xblock(const LayerPlan& L, unsigned flags)
{
    if (L.generic_passes || !mac_xb_available(L) || !fast_pass_available(L.d.Ny)) return false;
    return (flags & ZNNI_MAC_XBLOCK) != 0;
}

// Internal flag: the x axis is transformed at full length, the multiply-accumulate form is the library's choice.
constexpr unsigned ROUTE_FULL_X = 1u << 30;

// Whether a batch of small images goes untransformed along x with its z and y transforms done four planes at a time: two
// kernels around the multiply-accumulate where the fully transformed route has four, products on split halves instead of
// fp32.  Against that stand kx products per output column (of whole column tiles) instead of about one per bin.  So its
// products, at the rate its multiply-accumulate reaches, are held against the other form's spectrum values and the two x
// passes.  Over 452 random batches of 8 to 64 inputs that go here (lengths up to 64, up to 800 images, 1 to 9 taps) 1.38 times as
// fast as on the fully transformed route on average, the worst 5 % behind (22 x 198 -> 485 of 16 x 18 x 18, 5^3 kernels);
// 64 x 80 -> 80 of 51^3, 5^3 7.1 against 9.7 ms; 8 x 32 -> 32 of 64^3, 7^3 0.51 against 0.67.
// Fewer inputs go here where their transformed images are at most PLANES_SMALL together: what counts there are launches, and
// this route has two fewer than either other.  Against the other untransformed one that is all: over 1179 random layers 1.18
// times as fast, five more than 3 % behind (29 -> 3 of 70 x 49 x 51, 3^3 kernels 68 against 61 us), where a transform's
// workgroups are a few more than a multiple of the chip's 256 units.  The fully transformed one multiplies sixteen bins of a
// pencil at a time in workgroups of their own, where a wave here walks through the whole sum.  A step of four (quad, tap) slots
// costs it 0.34 us more with no row tiles to multiply and 0.11 less with each (the other form takes four steps for it), a
// chunk of sixteen images 0.59, 0.085 less with each input (x passes).  Two launches (8.4 us) and the quicker products of the
// second tap and the next ones (2.2 ps a value of the kernel bank) make up for it or not; where the batch form would serve all
// inputs, its products count as above.  Up to 96 images that is never much (1061 layers: 7 more than 5 % behind, the worst 17 %;
// 4 x 121 -> 3 of 11^3, 9 x 9 x 8 kernels 88 us here, 67 there), and the sums here are the closer ones (stepwise): always this
// route.  Over 2090 random layers of 1 to 7 inputs (lengths up to 64, 1 to 1500 images, 1 to 9 taps) 1.159 times as fast as on that
// route and 1.044 times as on this one, the better of the two 1.165 and 1.049; 62 more than 5 % off the better (7 x 227 -> 1460
// of 8^3, 2^3 kernels 353 us here, 262 there).  Always this route is as little as half as fast (1104 -> 2 of 8^3, 7^3 386 against
// 202), never as well (1061 -> 69 of 7^3, 5 x 4 x 4 402 against 659).
constexpr double PLANES_SMALL = 40e6;
static bool pick_planes(const LayerPlan& L, unsigned flags)
{
    if (flags & (ROUTE_FULL_X | ZNNI_MAC_REFERENCE | ZNNI_MAC_SINGLE | ZNNI_MAC_BATCH | ZNNI_MAC_XDIRECT | ZNNI_MAC_XBLOCK)) return false;
    if (!mac_xd_available(L) || !fused_planes_available(L)) return false;
    const Dims& d = L.d;
    const double pairs = (double)L.fp * L.Mp, pencils = (double)d.zc * d.Ny;
    // seconds of a pencil
    const double products = 24.0 * d.kx * ((d.nox + 15) & ~15) * pairs * L.S / MAC_SPLIT_FLOPS;
    const double batch = MAC_BATCH_SEC_PER_VALUE * pairs * d.Nx * ((L.S + 15) / 16);
    const double passes = 8.0 * ((double)L.nimg * (d.nx + d.Nx) + (double)L.nimgo * (d.Nx + d.nox)) / 5e12;
    if (L.S >= 8) return products < batch + passes;
    if (8.0 * (L.nimg + (double)L.nimgo) * d.nx * pencils > PLANES_SMALL) return false;
    if (pick_untransformed_x(L, flags)) return true;
    if (L.f <= 96) return true;
    double gain = 8.4e-6 - (0.59e-6 - 0.085e-6 * L.S) / 16 * L.f - (0.34e-6 - 0.11e-6 * L.mac_RTW) / 16 * d.kx * L.fp +
                  2.2e-12 * (d.kx - 1) * pairs * pencils;
    if (mac_batch_preferred(L) && products > batch + passes) gain -= 3.5 * (products - batch - passes) * pencils;
    return gain > 0;
}

static bool pick_xdirect(const LayerPlan& L, unsigned flags)
{
    if (L.xblock || L.planes) return true;
    if (flags & ROUTE_FULL_X) return false;
    if (L.generic_passes || !mac_xd_available(L) || !fast_pass_available(L.d.Ny)) return false;
    if (flags & ZNNI_MAC_XDIRECT) return true;
    if (flags & ZNNI_MAC_XBLOCK) return false;
    return pick_untransformed_x(L, flags);
}

// Shape part of a plan: validates, fills every size and the array sizes sz[]; assigns no pointers.
static znni_status shape_plan(int S, int f, int fo, const int n[3], const int k[3], unsigned flags, LayerPlan* L)
{
    if (!n || !k) return ZNNI_ERR_NULL;
    if (S < 1 || f < 1 || fo < 1) return ZNNI_ERR_SHAPE;
    for (int a = 0; a < 3; ++a)
        if (n[a] < 1 || k[a] < 1 || k[a] > n[a]) return ZNNI_ERR_SHAPE;
    Dims& d = L->d;
    d.nx = n[0]; d.ny = n[1]; d.nz = n[2];
    d.kx = k[0]; d.ky = k[1]; d.kz = k[2];
    d.Nx = fft_size(d.nx); d.Ny = fft_size(d.ny); d.Nz = fft_size(d.nz);
    if (d.Nx == 0 || d.Ny == 0 || d.Nz == 0) return ZNNI_ERR_UNSUPPORTED_SIZE;
    // launch-grid limits (grid y/z <= 65535) and 32-bit index products used inside the kernels
    if ((long long)S * f > 65535 || (long long)S * fo > 65535) return ZNNI_ERR_SHAPE;
    const int kmax = d.kx > d.ky ? (d.kx > d.kz ? d.kx : d.kz) : (d.ky > d.kz ? d.ky : d.kz);
    const int nmax = d.nx > d.ny ? (d.nx > d.nz ? d.nx : d.nz) : (d.ny > d.nz ? d.ny : d.nz);
    if (((long long)fo + 15) * (f + 3) * kmax * kmax > (1ll << 30)) return ZNNI_ERR_SHAPE;
    if ((long long)S * (f > fo ? f : fo) * nmax > (1ll << 30)) return ZNNI_ERR_SHAPE;
    L->S = S; L->f = f; L->fo = fo;
    d.zc = d.Nz / 2 + 1;
    d.nox = d.nx - d.kx + 1; d.noy = d.ny - d.ky + 1; d.noz = d.nz - d.kz + 1;
    d.ldy = (d.ny + 15) & ~15;       // X1, X2 and Y1 rows start on 128-byte boundaries
    d.ldx = (d.nx + 15) & ~15;
    d.ldo = (d.noy + 15) & ~15;
    // Y2 rows: padded to 128-byte boundaries only where they would not even start on 64-byte ones (lengths
    // like 100: the inverse x pass, which stores 128-byte runs into them, is then 20 % faster); where rows are
    // 64-byte aligned anyway the extra bytes cost more than the alignment gains (measured at 40 and 72)
    d.ldn = (d.Ny % 8 == 0) ? d.Ny : ((d.Ny + 15) & ~15);
    d.ldxo = (d.nox + 15) & ~15;
    L->nimg = S * f;
    L->nimgo = S * fo;
    L->fp = (f + 3) & ~3;
    plan_mac(L);        // also sets Mp
    L->tiles = false;
    L->generic_passes = (flags & ZNNI_PASSES_REFERENCE) != 0;
    L->xblock = pick_xblock(*L, flags);
    L->planes = pick_planes(*L, flags);
    L->xdirect = pick_xdirect(*L, flags);
    // X2 and Yd are ordered [image][oz][oy]; the order [oz][image][oy] was measured too: 2 % faster for the
    // multiply-accumulate that reads X2 and writes Yd, 6 % slower for the y passes on the other side of them
    d.x2i = d.zc * d.Ny; d.x2o = d.Ny;
    d.ydi = d.zc * d.Ny; d.ydo = d.Ny;
    make_fft_plan(d.Nx, &L->fftx);
    make_fft_plan(d.Ny, &L->ffty);
    make_fft_plan(d.Nz, &L->fftz);

    const size_t c = sizeof(float2);
    const size_t zc = d.zc, nimg = L->nimg, nimgo = L->nimgo;
    L->sz[0] = zc * d.ky * d.kx * L->fp * L->Mp * c;                                    // A1
    // A + room for the operand requests the multiply-accumulate issues one group of steps past the end
    L->sz[1] = zc * d.Ny * d.kx * L->fp * L->Mp * c + (size_t)(L->fp + 64) * L->Mp * c;
    if (mac_xb_available(*L) && mac_xb_kernel_bytes(*L) > L->sz[1]) L->sz[1] = mac_xb_kernel_bytes(*L);
    // Sized for either route (x axis transformed or not), so that the workspace a shape needs does not depend on
    // the flags of the call.
    size_t b0 = nimg * d.nx * zc * d.ldy;                            // X1
    size_t t = zc * d.Ny * nimg * d.Nx; if (t > b0) b0 = t;          // Xt
    t = nimgo * zc * d.nox * d.ldn; if (t > b0) b0 = t;              // Y2
    const size_t yd = nimgo * zc * d.Ny * d.ldxo;                    // Yd
    if (yd > b0) b0 = yd;
    size_t b1 = nimg * zc * d.Ny * d.ldx;                            // X2
    t = nimgo * d.nox * zc * d.ldo; if (t > b1) b1 = t;              // Y1
    L->sz[2] = b0 * c;
    L->sz[3] = b1 * c;
    t = zc * d.Ny * nimgo * d.Nx;                                    // Yt
    L->sz[4] = (t > yd ? t : yd) * c;
    return ZNNI_OK;
}

// Pointer part: carve the workspace at `base` into arrays of the given byte sizes.  own_yt = false: the output
// spectra share buf1 (a whole-layer call never needs X2 or Y1 while Yt is alive), or buf0 where the x axis is not
// transformed (X1 is dead by then and X2, in buf1, is being read).
static void place_plan(LayerPlan* L, void* base, const size_t sz[5], bool own_yt)
{
    const Dims& d = L->d;
    const size_t c = sizeof(float2);
    size_t off = 0;
    // addresses as integers: a size query carves from a null base
    const uintptr_t p = (uintptr_t)base;
    L->twx = (float2*)(p + off); off += align_up((size_t)d.Nx * c, 256);
    L->twy = (float2*)(p + off); off += align_up((size_t)d.Ny * c, 256);
    L->twz = (float2*)(p + off); off += align_up((size_t)d.Nz * c, 256);
    L->A1 = (float2*)(p + off); off += align_up(sz[0], 256);
    L->A = (float2*)(p + off); off += align_up(sz[1], 256);
    // behind the stored transforms, where the other routes' kernels read their padding
    L->rs = (float*)(L->A + (size_t)d.zc * d.Ny * d.kx * L->fp * L->Mp);
    L->oz0 = 0; L->ozn = d.zc;
    L->buf0 = (float2*)(p + off); off += align_up(sz[2], 256);
    // (sz[2] already covers Yd, so nothing is added for the layers whose x axis is not transformed)
    const size_t b1 = own_yt ? sz[3] : (sz[3] > sz[4] ? sz[3] : sz[4]);
    L->buf1 = (float2*)(p + off); off += align_up(b1, 256);
    if (own_yt) { L->Yt = (float2*)(p + off); off += align_up(sz[4], 256); }
    else L->Yt = L->xdirect ? L->buf0 : L->buf1;
    L->bytes = off;
}

znni_status make_whole_plan(int S, int f, int fo, const int n[3], const int k[3], unsigned flags, void* base, LayerPlan* L)
{
    znni_status rc = shape_plan(S, f, fo, n, k, flags, L);
    if (rc) return rc;
    place_plan(L, base, L->sz, false);
    return ZNNI_OK;
}

// Tiles are for calls that name no form and no passes.
static bool may_tile(unsigned flags) { return !(flags & ~(unsigned)(ZNNI_RELU | ZNNI_KEEP_KERNELS)); }

znni_status make_plan(int S, int f, int fo, const int n[3], const int k[3], unsigned flags, void* base,
                      LayerPlan* L)
{
    znni_status rc = make_whole_plan(S, f, fo, n, k, flags, base, L);
    if (rc) return rc;
    // (the workspace stays what a shape needs on any route)
    if (may_tile(flags))
        if (const int N = pick_tiles(*L, L->bytes, false)) tiles_plan(*L, N, base, L->bytes, false, L);
    return ZNNI_OK;
}

// ------------------------------------------------------------------------------------------- sub-layers
// Section VII-A: a layer of shape (S, f, f') can be computed as sub-layers of shapes (S_i, f_i, f'_i), each small
// enough for the memory at hand.  Here the memory at hand is the caller's workspace.  The division follows the
// paper's preference: whole-layer if it fits; else sub-batches (f_i = f, f'_i = f', S_i < S), which transform
// every input and output once; else S_i = 1 with blocks of f_a input and f'_a output images.  In the last case
// the sub-layers of one output block accumulate their products in the output spectra (kept in a buffer of their
// own), so each output block is inverse-transformed once, and the input transforms are repeated once per output
// block.
struct Division {
    int Si, fi, foi;
    bool own_yt;
    size_t sz[5];
    size_t bytes;
};

// Workspace of a division: arrays sized for its largest sub-layer (the ragged last chunks are smaller).
static znni_status division_bytes(int S, int f, int fo, const int n[3], const int k[3], Division* D)
{
    D->own_yt = D->fi < f;
    for (int q = 0; q < 5; ++q) D->sz[q] = 0;
    // distinct sub-layer shapes: full or ragged in each of S, f, f'
    const int Ss[2] = {D->Si, S % D->Si}, fs[2] = {D->fi, f % D->fi}, fos[2] = {D->foi, fo % D->foi};
    LayerPlan L;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b)
            for (int c = 0; c < 2; ++c) {
                if (Ss[a] == 0 || fs[b] == 0 || fos[c] == 0) continue;
                znni_status rc = shape_plan(Ss[a], fs[b], fos[c], n, k, 0, &L);
                if (rc) return rc;
                for (int q = 0; q < 5; ++q)
                    if (L.sz[q] > D->sz[q]) D->sz[q] = L.sz[q];
            }
    place_plan(&L, nullptr, D->sz, D->own_yt);
    D->bytes = L.bytes;
    return ZNNI_OK;
}

// Rough HBM traffic of a division in units of one transformed image (what the choice between blockings is
// based on): three forward passes per input image and output block, one read-modify-write of the output spectra
// per input block, three inverse passes per output image.
static double division_cost(int f, int fo, int fi, int foi)
{
    const double nfo = (fo + foi - 1) / foi, nfi = (f + fi - 1) / fi;
    return 5.0 * f * nfo + 2.0 * fo * (nfi - 1) + 5.0 * fo;
}

static znni_status choose_division(int S, int f, int fo, const int n[3], const int k[3], size_t budget,
                                   Division* D)
{
    if (!n || !k) return ZNNI_ERR_NULL;
    if (S < 1 || f < 1 || fo < 1) return ZNNI_ERR_SHAPE;
    D->Si = S; D->fi = f; D->foi = fo;
    znni_status rc = division_bytes(S, f, fo, n, k, D);
    if (rc) return rc;
    if (D->bytes <= budget) return ZNNI_OK;
    // sub-batches: the largest S_i that fits
    if (S > 1) {
        int lo = 0, hi = S;             // lo fits (0 = none), hi does not
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            D->Si = mid;
            rc = division_bytes(S, f, fo, n, k, D);
            if (rc) return rc;
            if (D->bytes <= budget) lo = mid; else hi = mid;
        }
        if (lo >= 1) {
            D->Si = lo;
            return division_bytes(S, f, fo, n, k, D);
        }
    }
    // blocks of input and output images, one input at a time: input blocks of f, then multiples of 4 (the
    // matrix-core contraction step), then 2 and 1; output blocks of f', then multiples of 16 (the matrix-core
    // tile), then 8, 4, 2, 1
    D->Si = 1;
    Division best;
    double best_cost = -1.0;
    auto next = [](int cur, int full, int step) {
        if (cur > step) return cur == full && full % step ? full / step * step : cur - step;
        return cur / 2;                 // step, step/2, ..., 1, 0
    };
    for (int foi = fo; foi >= 1; foi = next(foi, fo, 16)) {
        // the largest input block that fits with this output block
        int fit = 0;
        for (int fi = f; fi >= 1; fi = next(fi, f, 4)) {
            D->fi = fi; D->foi = foi;
            rc = division_bytes(S, f, fo, n, k, D);
            if (rc) return rc;
            if (D->bytes <= budget) { fit = fi; break; }
        }
        if (fit) {
            const double cost = division_cost(f, fo, fit, foi);
            if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = *D; }
        }
    }
    if (best_cost < 0) return ZNNI_ERR_WORKSPACE;
    *D = best;
    return ZNNI_OK;
}

// Known bits only, and at most one of the three bits that pick a multiply-accumulate form.
static bool flags_ok(unsigned flags)
{
    const unsigned all_forms = ZNNI_MAC_REFERENCE | ZNNI_MAC_SINGLE | ZNNI_MAC_BATCH | ZNNI_MAC_XDIRECT | ZNNI_MAC_XBLOCK;
    if (flags & ~(unsigned)(ZNNI_RELU | ZNNI_KEEP_KERNELS | ZNNI_PASSES_REFERENCE | all_forms)) return false;
    const unsigned forms = flags & all_forms;
    return (forms & (forms - 1)) == 0;
}

static znni_status validate(int S, int f, int fo, const int n[3], const int k[3], const float* in,
                            const float* w, float* out, unsigned flags, void* workspace,
                            size_t workspace_bytes, LayerPlan* L)
{
    if (!in || !w || !out || !workspace) return ZNNI_ERR_NULL;
    if (!flags_ok(flags)) return ZNNI_ERR_FLAGS;
    znni_status rc = make_plan(S, f, fo, n, k, flags, workspace, L);
    if (rc) return rc;
    if (((uintptr_t)in | (uintptr_t)w | (uintptr_t)out) & 15u) return ZNNI_ERR_ALIGN;
    if ((uintptr_t)workspace & 255u) return ZNNI_ERR_ALIGN;
    if (workspace_bytes < L->bytes) return ZNNI_ERR_WORKSPACE;
    return ZNNI_OK;
}

#define ZNNI_DO(call)          \
    do {                       \
        rc = (call);           \
        if (rc) return rc;     \
    } while (0)

// The transforms before and after the multiply-accumulate of a layer whose x axis is not transformed.
static znni_status fwd_untransformed_x(const LayerPlan& L, const float* in, hipStream_t st)
{
    if (L.planes) return launch_fwd_zy_planes(L, in, nullptr, st);
    const znni_status rc = launch_fwd_z(L, in, st);
    return rc ? rc : launch_fwd_y(L, st);
}
static znni_status inv_untransformed_x(const LayerPlan& L, const float* bias, float* out, unsigned flags, hipStream_t st)
{
    if (L.planes) return launch_inv_yz_planes(L, bias, out, flags, st);
    const znni_status rc = launch_fast_inv_yt(L, st);
    return rc ? rc : launch_inv_z(L, bias, out, flags, st);
}

// Runs the stages in order; if ev != NULL records ev[s] before stage s and ev[ZNNI_NUM_STAGES] at the end.
static znni_status run(const LayerPlan& L, const float* in, const float* w, const float* bias, float* out,
                       unsigned flags, hipStream_t st, hipEvent_t* ev)
{
    znni_status rc;
#define ZNNI_MARK(s)                                                          \
    do {                                                                      \
        if (ev && hipEventRecord(ev[s], st) != hipSuccess) return ZNNI_ERR_HIP; \
    } while (0)
    const size_t bank = (size_t)L.f * L.d.kx * L.d.ky * L.d.kz;
    if (!ev && !(flags & ZNNI_KEEP_KERNELS) && prep_small_available(L)) {
        // four launches instead of six (with events between the stages: six, and the same results)
        ZNNI_DO(launch_fwd_zy_planes(L, in, w, st));
        ZNNI_DO(launch_kernel_prep_y(L, st));
        ZNNI_DO(launch_mac_xd(L, 0, st));
        return launch_inv_yz_planes(L, bias, out, flags, st);
    }
    ZNNI_DO(launch_twiddles(L, flags & ZNNI_KEEP_KERNELS ? nullptr : w, bank, st));
    ZNNI_MARK(ZNNI_STAGE_KERNEL_PREP);
    // the stored kernel transforms of an earlier call on this workspace may be kept (same w, shape and form)
    if (!(flags & ZNNI_KEEP_KERNELS)) ZNNI_DO(launch_kernel_prep(L, w, bank, st));
    if (L.tiles && (L.cut.sn < L.cut.S || L.cut.pn < L.cut.pairs)) {
        // tile pairs take turns (under a budget only)
        if (ev) return ZNNI_ERR_WORKSPACE;
        LayerPlan T = L;
        auto& c = T.cut;
        for (c.s0 = 0; c.s0 < c.S; c.s0 += L.cut.sn)
            for (c.p0 = 0; c.p0 < c.pairs; c.p0 += L.cut.pn) {
                c.sn = c.S - c.s0 < L.cut.sn ? c.S - c.s0 : L.cut.sn;
                c.pn = c.pairs - c.p0 < L.cut.pn ? c.pairs - c.p0 : L.cut.pn;
                T.S = c.sn * c.pn; T.nimg = T.S * T.f; T.nimgo = T.S * T.fo;
                ZNNI_DO(launch_fwd_zy_planes(T, in, nullptr, st));
                ZNNI_DO(launch_mac_xd(T, 0, st));
                ZNNI_DO(launch_inv_yz_planes(T, bias, out, flags, st));
            }
        return ZNNI_OK;
    }
    if (L.xdirect) {
        // x axis not transformed: the x stages do nothing and read about zero
        ZNNI_MARK(ZNNI_STAGE_FWD_Z);
        ZNNI_DO(L.planes ? launch_fwd_zy_planes(L, in, nullptr, st) : launch_fwd_z(L, in, st));
        ZNNI_MARK(ZNNI_STAGE_FWD_Y);
        if (!L.planes) ZNNI_DO(launch_fwd_y(L, st));
        ZNNI_MARK(ZNNI_STAGE_FWD_X);
        ZNNI_MARK(ZNNI_STAGE_MAC);
        ZNNI_DO(L.xblock ? launch_mac_xb(L, 0, st) : launch_mac_xd(L, 0, st));
        ZNNI_MARK(ZNNI_STAGE_INV_X);
        ZNNI_MARK(ZNNI_STAGE_INV_Y);
        ZNNI_DO(L.planes ? launch_inv_yz_planes(L, bias, out, flags, st) : launch_fast_inv_yt(L, st));
        ZNNI_MARK(ZNNI_STAGE_INV_Z);
        if (!L.planes) ZNNI_DO(launch_inv_z(L, bias, out, flags, st));
        ZNNI_MARK(ZNNI_NUM_STAGES);
        return ZNNI_OK;
    }
    const bool fused_zy = fused_fwd_zy_available(L);       // then the z stage's time covers z and y
    ZNNI_MARK(ZNNI_STAGE_FWD_Z);
    if (fused_zy) ZNNI_DO(launch_fwd_zy(L, in, st));
    else ZNNI_DO(launch_fwd_z(L, in, st));
    ZNNI_MARK(ZNNI_STAGE_FWD_Y);
    if (!fused_zy) ZNNI_DO(launch_fwd_y(L, st));
    ZNNI_MARK(ZNNI_STAGE_FWD_X);
    if (fused_zy) ZNNI_DO(launch_fast_fwd_xt(L, st));
    else ZNNI_DO(launch_fwd_x(L, st));
    ZNNI_MARK(ZNNI_STAGE_MAC);
    ZNNI_DO(launch_mac(L, flags, 0, st));
    ZNNI_MARK(ZNNI_STAGE_INV_X);
    ZNNI_DO(launch_inv_x(L, st));
    const bool fused_yz = fused_inv_yz_available(L);       // then the y stage's time covers both
    ZNNI_MARK(ZNNI_STAGE_INV_Y);
    if (fused_yz) ZNNI_DO(launch_inv_yz(L, bias, out, flags, st));
    else ZNNI_DO(launch_inv_y(L, st));
    ZNNI_MARK(ZNNI_STAGE_INV_Z);
    if (!fused_yz) ZNNI_DO(launch_inv_z(L, bias, out, flags, st));
    ZNNI_MARK(ZNNI_NUM_STAGES);
#undef ZNNI_MARK
    return ZNNI_OK;
}

// Flags that give every block of input images of an output block the same route.  Their products are added up in one
// set of output spectra, whose layout is the route's; the rules that pick a route look at the number of input images, so
// the last, smaller block, planned by itself, can come out differently from the others (91 -> 38 images of 18^3, 6^3
// kernels in blocks of 68).  The full blocks decide; a form of theirs that the last block does not have (blocks of eight
// along x under 16 images) counts as one that does not exist.
static unsigned one_route(int S, int f, int fi, int fo, const int n[3], const int k[3], unsigned flags)
{
    if (fi >= f || f % fi == 0) return flags;
    LayerPlan full, rest;
    if (shape_plan(S, fi, fo, n, k, flags, &full) || shape_plan(S, f % fi, fo, n, k, flags, &rest)) return flags;
    if (full.xblock != rest.xblock) return (flags & ~(unsigned)ZNNI_MAC_XBLOCK) | ROUTE_FULL_X;
    if (full.xdirect != rest.xdirect) return flags | (full.xdirect ? (unsigned)ZNNI_MAC_XDIRECT : ROUTE_FULL_X);
    if (full.planes != rest.planes) return flags | (unsigned)ZNNI_MAC_XDIRECT;
    return flags;
}

// The layer as the sub-layers of division D, all on one workspace.
static znni_status run_divided(const Division& D, int S, int f, int fo, const int n[3], const int k[3],
                               const float* in, const float* w, const float* bias, float* out, unsigned flags,
                               void* workspace, hipStream_t st)
{
    znni_status rc;
    const size_t nvox = (size_t)n[0] * n[1] * n[2], kvol = (size_t)k[0] * k[1] * k[2];
    const size_t ovox = (size_t)(n[0] - k[0] + 1) * (n[1] - k[1] + 1) * (n[2] - k[2] + 1);
    for (int s0 = 0; s0 < S; s0 += D.Si) {
        const int Sc = S - s0 < D.Si ? S - s0 : D.Si;
        for (int j0 = 0; j0 < fo; j0 += D.foi) {
            const int foc = fo - j0 < D.foi ? fo - j0 : D.foi;
            const unsigned route = one_route(Sc, f, D.fi, foc, n, k, flags);
            LayerPlan L;
            for (int i0 = 0; i0 < f; i0 += D.fi) {
                const int fc = f - i0 < D.fi ? f - i0 : D.fi;
                // a block of images is one contiguous tensor only if it spans all images of a tuple or one tuple
                if (Sc > 1 && (fc != f || foc != fo)) return ZNNI_ERR_SHAPE;
                ZNNI_DO(shape_plan(Sc, fc, foc, n, k, route, &L));
                for (int q = 0; q < 5; ++q)
                    if (L.sz[q] > D.sz[q]) return ZNNI_ERR_WORKSPACE;
                place_plan(&L, workspace, D.sz, D.own_yt);
                const float* wsub = w + ((size_t)j0 * f + i0) * kvol;
                ZNNI_DO(launch_twiddles(L, wsub, (size_t)f * kvol, st));      // also zeroes the padding behind this chunk's A
                ZNNI_DO(launch_kernel_prep(L, wsub, (size_t)f * kvol, st));
                const float* isub = in + ((size_t)s0 * f + i0) * nvox;
                if (L.xdirect) {
                    ZNNI_DO(fwd_untransformed_x(L, isub, st));
                    ZNNI_DO(L.xblock ? launch_mac_xb(L, i0 > 0, st) : launch_mac_xd(L, i0 > 0, st));
                    continue;
                }
                if (fused_fwd_zy_available(L)) {
                    ZNNI_DO(launch_fwd_zy(L, isub, st));
                    ZNNI_DO(launch_fast_fwd_xt(L, st));
                } else {
                    ZNNI_DO(launch_fwd_z(L, isub, st));
                    ZNNI_DO(launch_fwd_y(L, st));
                    ZNNI_DO(launch_fwd_x(L, st));
                }
                ZNNI_DO(launch_mac(L, route, i0 > 0, st));
            }
            const float* bsub = bias ? bias + j0 : nullptr;
            float* osub = out + ((size_t)s0 * fo + j0) * ovox;
            if (L.xdirect) {
                ZNNI_DO(inv_untransformed_x(L, bsub, osub, flags, st));
                continue;
            }
            ZNNI_DO(launch_inv_x(L, st));
            if (fused_inv_yz_available(L)) {
                ZNNI_DO(launch_inv_yz(L, bsub, osub, flags, st));
            } else {
                ZNNI_DO(launch_inv_y(L, st));
                ZNNI_DO(launch_inv_z(L, bsub, osub, flags, st));
            }
        }
    }
    return ZNNI_OK;
}

// A whole layer whose kernel transforms do not fit: everything as in a whole-layer call, but the second stage of the
// kernel transform and the multiply-accumulate go through the rows of the halved axis in slabs that share one piece of
// memory.  Nothing is transformed twice, so this is taken before any division of the images (48 -> 48 images of 160^3,
// 5^3 kernels with half the workspace: blocks of images 4.64 ms, slabs 2.7 ms; in turns of tiles, which come first where the whole
// layer takes tiles, 1.7).  The result is that of the whole-layer call through whole planes, bit for bit.  Only the routes that do not transform x (their kernel transforms lie row by row), and only slabs of
// at least SLAB_PENCILS pencils: smaller ones would leave the chip idle between them.
constexpr int SLAB_PENCILS = 512;
static bool plan_slabs(int S, int f, int fo, const int n[3], const int k[3], unsigned flags, void* workspace,
                       size_t budget, LayerPlan* L, int* rows)
{
    if (shape_plan(S, f, fo, n, k, flags, L) || !L->xdirect) return false;
    const Dims& d = L->d;
    const size_t row = L->xblock ? mac_xb_kernel_bytes(*L) / d.zc
                                 : (size_t)d.Ny * d.kx * L->fp * L->Mp * sizeof(float2);
    size_t sz[5] = {L->sz[0], 0, L->sz[2], L->sz[3], 0};       // no Yt of its own: Yd takes turns with X1 in buf0
    place_plan(L, workspace, sz, false);
    const size_t scales = align_up(split_scale_floats(*L) * sizeof(float), 256);
    if (budget < L->bytes + scales + 256) return false;
    *rows = (int)((budget - L->bytes - scales - 256) / row < (size_t)d.zc ? (budget - L->bytes - scales - 256) / row : d.zc);
    if ((long long)*rows * d.Ny < SLAB_PENCILS) return false;
    *rows = (d.zc + (d.zc + *rows - 1) / *rows - 1) / ((d.zc + *rows - 1) / *rows);      // slabs of about the same size
    sz[1] = scales + (size_t)*rows * row;
    place_plan(L, workspace, sz, false);
    L->rs = (float*)L->A;
    L->A = (float2*)((uintptr_t)L->A + scales);
    return L->bytes <= budget;
}

static znni_status run_slabs(LayerPlan L, int rows, const float* in, const float* w, const float* bias, float* out,
                             unsigned flags, hipStream_t st)
{
    znni_status rc;
    const size_t bank = (size_t)L.f * L.d.kx * L.d.ky * L.d.kz;
    ZNNI_DO(launch_twiddles(L, w, bank, st));
    ZNNI_DO(launch_kernel_prep_z(L, w, bank, st));
    ZNNI_DO(fwd_untransformed_x(L, in, st));
    for (L.oz0 = 0; L.oz0 < L.d.zc; L.oz0 += rows) {
        L.ozn = L.d.zc - L.oz0 < rows ? L.d.zc - L.oz0 : rows;
        ZNNI_DO(launch_kernel_prep_y(L, st));
        ZNNI_DO(L.xblock ? launch_mac_xb(L, 0, st) : launch_mac_xd(L, 0, st));
    }
    return inv_untransformed_x(L, bias, out, flags, st);
}

// Bytes and flops of every stage of a plan (znni_conv3d_fft_stage_work_v, znni_conv3d_fft_call_work_v).
void plan_work(const LayerPlan& L, unsigned flags, double hbm_bytes[ZNNI_NUM_STAGES], double flops[ZNNI_NUM_STAGES])
{
    const Dims& d = L.d;
    const double c = sizeof(float2), ni = L.nimg, no = L.nimgo, zc = d.zc;
    const double vox = (double)d.nx * d.ny * d.nz, ovox = (double)d.nox * d.noy * d.noz;
    const double x1 = c * d.nx * d.ny * zc, x2 = c * d.nx * d.Ny * zc, xt = c * (double)d.Nx * d.Ny * zc;
    const double y2 = c * zc * d.nox * d.Ny, y1 = c * (double)d.nox * d.noy * zc;
    // stored kernel transforms, unpadded: kx values per kernel column along x, or 8 where x goes in blocks of eight
    const double a = c * zc * d.Ny * (double)L.f * L.fo * (L.xblock ? 8 : d.kx);
    for (int q = 0; q < ZNNI_NUM_STAGES; ++q) hbm_bytes[q] = flops[q] = 0.0;
    if (L.tiles) {
        // pairs of tiles: whole complex planes [Nz][Ny], whichever take turns
        const auto& t = L.cut;
        const double in = (double)t.S * L.f * d.nx, out = (double)t.S * L.fo * d.nox, plane = (double)t.pairs * d.Ny * d.Nz;
        if (!(flags & ZNNI_KEEP_KERNELS)) hbm_bytes[ZNNI_STAGE_KERNEL_PREP] = 4.0 * L.f * L.fo * d.kx * d.ky * d.kz + a;
        hbm_bytes[ZNNI_STAGE_FWD_Z] = in * (4.0 * t.ny * t.nz + c * plane);
        hbm_bytes[ZNNI_STAGE_MAC] = c * plane * (in + out) + a;
        hbm_bytes[ZNNI_STAGE_INV_Y] = out * (c * plane + 4.0 * t.noy * t.noz);
        flops[ZNNI_STAGE_MAC] = 8.0 * d.kx * L.f * plane * out;
        return;
    }
    if (!(flags & ZNNI_KEEP_KERNELS)) hbm_bytes[ZNNI_STAGE_KERNEL_PREP] = 4.0 * L.f * L.fo * d.kx * d.ky * d.kz + a;
    const bool fused_zy = L.planes || (!L.xdirect && fused_fwd_zy_available(L)), fused_yz = L.planes || (!L.xdirect && fused_inv_yz_available(L));
    if (fused_zy) hbm_bytes[ZNNI_STAGE_FWD_Z] = ni * (4.0 * vox + x2);
    else {
        hbm_bytes[ZNNI_STAGE_FWD_Z] = ni * (4.0 * vox + x1);
        hbm_bytes[ZNNI_STAGE_FWD_Y] = ni * (x1 + x2);
    }
    if (fused_yz) hbm_bytes[ZNNI_STAGE_INV_Y] = no * (y2 + 4.0 * ovox);
    else {
        hbm_bytes[ZNNI_STAGE_INV_Y] = no * (y2 + y1);
        hbm_bytes[ZNNI_STAGE_INV_Z] = no * (y1 + 4.0 * ovox);
    }
    if (L.xdirect) {
        // the spectra between the y passes and the multiply-accumulate keep the x axis as it is
        const double bins = zc * d.Ny * d.nox;
        hbm_bytes[ZNNI_STAGE_MAC] = ni * x2 + a + no * y2;
        flops[ZNNI_STAGE_MAC] = 8.0 * d.kx * L.S * (double)L.f * L.fo * bins;
        if (L.xblock) {
            // one length-8 product per block of V = 9 - kx outputs
            const int V = 9 - d.kx;
            flops[ZNNI_STAGE_MAC] = 8.0 * 8 * L.S * (double)L.f * L.fo * zc * d.Ny * ((d.nox + V - 1) / V);
        }
    } else {
        const double bins = zc * d.Ny * d.Nx;
        hbm_bytes[ZNNI_STAGE_FWD_X] = ni * (x2 + xt);
        hbm_bytes[ZNNI_STAGE_INV_X] = no * (xt + y2);
        hbm_bytes[ZNNI_STAGE_MAC] = ni * xt + a + no * xt;
        flops[ZNNI_STAGE_MAC] = (8.0 * L.S + 8.0 * (d.kx - 1)) * (double)L.f * L.fo * bins;
    }
}

// Device address of `scratch` on the current GPU, looked up once per GPU (each GPU holds its own copy of the
// array at its own address).
static znni_status static_scratch(void** out)
{
    constexpr int kMaxDevices = 64;
    static void* ptr[kMaxDevices];          // zero-initialised
    static std::mutex mu;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ZNNI_ERR_HIP;
    std::lock_guard<std::mutex> guard(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ZNNI_ERR_HIP;
        if ((uintptr_t)p & 255u) return ZNNI_ERR_ALIGN;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return ZNNI_OK;
}

// One 16-byte element per thread and as many workgroups as that takes: the launch shape that moved the most bytes
// per second of those tried (6.2 TB/s on 6 GiB; 8 elements per thread 5.3, grid-stride loops of 1024 to 4096
// workgroups 4.8 to 5.1, hipMemcpyAsync 4.5).
__global__ __launch_bounds__(256) void k_copy_probe(float4* __restrict__ dst, const float4* __restrict__ src, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

}  // namespace znni

using namespace znni;

extern "C" {

int znni_version(void) { return 200; }

const char* znni_status_string(int st)
{
    switch (st) {
        case ZNNI_OK: return "ok";
        case ZNNI_ERR_NULL: return "a required pointer is NULL";
        case ZNNI_ERR_SHAPE: return "bad layer shape (need S,f,f' >= 1 and 1 <= k <= n on every axis, counts within launch limits)";
        case ZNNI_ERR_UNSUPPORTED_SIZE: return "no supported transform size for this image edge";
        case ZNNI_ERR_WORKSPACE: return "workspace too small";
        case ZNNI_ERR_FLAGS: return "unknown flag bit, or more than one multiply-accumulate form requested";
        case ZNNI_ERR_HIP: return "HIP call or kernel launch failed";
        case ZNNI_ERR_ALIGN: return "device pointer not sufficiently aligned";
    }
    return "unknown status";
}

int znni_fft_size(int n) { return fft_size(n); }

znni_status znni_conv3d_fft_workspace_v(int S, int f, int fo, const int n[3], const int k[3], size_t* bytes)
{
    if (!bytes) return ZNNI_ERR_NULL;
    LayerPlan L;
    znni_status rc = make_plan(S, f, fo, n, k, 0, nullptr, &L);
    if (rc) return rc;
    *bytes = L.bytes;
    return ZNNI_OK;
}

znni_status znni_conv3d_fft_v(int S, int f, int fo, const int n[3], const int k[3], const float* in,
                              const float* w, const float* bias, float* out, unsigned flags, void* workspace,
                              size_t workspace_bytes, void* stream)
{
    LayerPlan L;
    znni_status rc = validate(S, f, fo, n, k, in, w, out, flags, workspace, workspace_bytes, &L);
    if (rc) return rc;
    return run(L, in, w, bias, out, flags, (hipStream_t)stream, nullptr);
}

static znni_status plan_and_work(decltype(make_plan)* plan, int S, int f, int fo, const int n[3], const int k[3], unsigned flags,
                                 double* hbm_bytes, double* flops)
{
    if (!hbm_bytes || !flops) return ZNNI_ERR_NULL;
    if (!flags_ok(flags)) return ZNNI_ERR_FLAGS;
    LayerPlan L;
    const znni_status rc = plan(S, f, fo, n, k, flags, nullptr, &L);
    if (rc) return rc;
    plan_work(L, flags, hbm_bytes, flops);
    return ZNNI_OK;
}

znni_status znni_conv3d_fft_stage_work_v(int S, int f, int fo, const int n[3], const int k[3], unsigned flags,
                                         double hbm_bytes[ZNNI_NUM_STAGES], double flops[ZNNI_NUM_STAGES])
{
    return plan_and_work(make_whole_plan, S, f, fo, n, k, flags, hbm_bytes, flops);
}

znni_status znni_conv3d_fft_call_work_v(int S, int f, int fo, const int n[3], const int k[3], unsigned flags,
                                        double hbm_bytes[ZNNI_NUM_STAGES], double flops[ZNNI_NUM_STAGES])
{
    return plan_and_work(make_plan, S, f, fo, n, k, flags, hbm_bytes, flops);
}

znni_status znni_conv3d_fft_static_v(int S, int f, int fo, const int n[3], const int k[3], const float* in,
                                     const float* w, const float* bias, float* out, unsigned flags, void* stream)
{
    // host-only checks first, against a stand-in workspace address (only its alignment matters to them)
    LayerPlan L;
    znni_status rc = validate(S, f, fo, n, k, in, w, out, flags, (void*)(uintptr_t)256, ZNNI_STATIC_SCRATCH_BYTES, &L);
    if (rc) return rc;                       // ZNNI_ERR_WORKSPACE: the layer needs more than the array holds
    void* base = nullptr;
    rc = static_scratch(&base);
    if (rc) return rc;
    rc = make_plan(S, f, fo, n, k, flags, base, &L);
    if (rc) return rc;
    return run(L, in, w, bias, out, flags, (hipStream_t)stream, nullptr);
}

znni_status znni_conv3d_fft_profile_v(int S, int f, int fo, const int n[3], const int k[3], const float* in,
                                      const float* w, const float* bias, float* out, unsigned flags,
                                      void* workspace, size_t workspace_bytes, void* stream, float* stage_ms)
{
    if (!stage_ms) return ZNNI_ERR_NULL;
    LayerPlan L;
    znni_status rc = validate(S, f, fo, n, k, in, w, out, flags, workspace, workspace_bytes, &L);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev[ZNNI_NUM_STAGES + 1];
    int made = 0;
    for (; made <= ZNNI_NUM_STAGES; ++made)
        if (hipEventCreate(&ev[made]) != hipSuccess) break;
    if (made <= ZNNI_NUM_STAGES) rc = ZNNI_ERR_HIP;
    if (!rc) rc = run(L, in, w, bias, out, flags, st, ev);
    if (!rc && hipStreamSynchronize(st) != hipSuccess) rc = ZNNI_ERR_HIP;
    if (!rc)
        for (int s = 0; s < ZNNI_NUM_STAGES; ++s)
            if (hipEventElapsedTime(&stage_ms[s], ev[s], ev[s + 1]) != hipSuccess) rc = ZNNI_ERR_HIP;
    for (int e = 0; e < made; ++e) (void)hipEventDestroy(ev[e]);
    return rc;
}

znni_status znni_conv3d_fft_workspace(int S, int f, int fo, int n, int k, size_t* bytes)
{
    const int nn[3] = {n, n, n}, kk[3] = {k, k, k};
    return znni_conv3d_fft_workspace_v(S, f, fo, nn, kk, bytes);
}

znni_status znni_conv3d_fft(int S, int f, int fo, int n, int k, const float* in, const float* w,
                            const float* bias, float* out, unsigned flags, void* workspace,
                            size_t workspace_bytes, void* stream)
{
    const int nn[3] = {n, n, n}, kk[3] = {k, k, k};
    return znni_conv3d_fft_v(S, f, fo, nn, kk, in, w, bias, out, flags, workspace, workspace_bytes, stream);
}

znni_status znni_conv3d_fft_profile(int S, int f, int fo, int n, int k, const float* in, const float* w,
                                    const float* bias, float* out, unsigned flags, void* workspace,
                                    size_t workspace_bytes, void* stream, float* stage_ms)
{
    const int nn[3] = {n, n, n}, kk[3] = {k, k, k};
    return znni_conv3d_fft_profile_v(S, f, fo, nn, kk, in, w, bias, out, flags, workspace, workspace_bytes,
                                     stream, stage_ms);
}

znni_status znni_conv3d_fft_sublayers_v(int S, int f, int fo, const int n[3], const int k[3],
                                        size_t budget_bytes, int sub[3], size_t* bytes)
{
    if (!sub || !bytes) return ZNNI_ERR_NULL;
    Division D;
    znni_status rc = choose_division(S, f, fo, n, k, budget_bytes, &D);
    if (rc == ZNNI_ERR_WORKSPACE) {
        // report what the smallest division would need
        D.Si = 1; D.fi = 1; D.foi = 1;
        if (division_bytes(S, f, fo, n, k, &D) == ZNNI_OK) *bytes = D.bytes;
        return rc;
    }
    if (rc) return rc;
    sub[0] = D.Si; sub[1] = D.fi; sub[2] = D.foi;
    *bytes = D.bytes;
    return ZNNI_OK;
}

znni_status znni_conv3d_fft_budget_v(int S, int f, int fo, const int n[3], const int k[3], const float* in,
                                     const float* w, const float* bias, float* out, unsigned flags,
                                     void* workspace, size_t workspace_bytes, void* stream)
{
    if (!in || !w || !out || !workspace) return ZNNI_ERR_NULL;
    // sub-layers take turns in the workspace, so there are no stored kernel transforms to keep between calls
    if (!flags_ok(flags) || (flags & ZNNI_KEEP_KERNELS)) return ZNNI_ERR_FLAGS;
    Division D;
    znni_status rc = choose_division(S, f, fo, n, k, workspace_bytes, &D);
    if (rc) return rc;
    if (((uintptr_t)in | (uintptr_t)w | (uintptr_t)out) & 15u) return ZNNI_ERR_ALIGN;
    if ((uintptr_t)workspace & 255u) return ZNNI_ERR_ALIGN;
    LayerPlan L;
    if (may_tile(flags)) {
        // Where the whole layer goes in tiles: they take less room, and their pairs can take turns in it.  The whole layer's
        // length, and so its result, where that fits.
        rc = make_whole_plan(S, f, fo, n, k, flags, nullptr, &L);
        if (rc) return rc;
        LayerPlan T;
        const int N = pick_tiles(L, L.bytes, false);
        L.bytes = workspace_bytes;
        if (N && (tiles_plan(L, N, workspace, workspace_bytes, true, &T) ||
                  tiles_plan(L, pick_tiles(L, workspace_bytes, true), workspace, workspace_bytes, true, &T)))
            return run(T, in, w, bias, out, flags, (hipStream_t)stream, nullptr);
    }
    if (D.Si < S || D.fi < f || D.foi < fo) {
        int rows = 0;
        if (plan_slabs(S, f, fo, n, k, flags, workspace, workspace_bytes, &L, &rows))
            return run_slabs(L, rows, in, w, bias, out, flags, (hipStream_t)stream);
    }
    return run_divided(D, S, f, fo, n, k, in, w, bias, out, flags, workspace, (hipStream_t)stream);
}

znni_status znni_copy_probe(void* dst, const void* src, size_t bytes, void* stream)
{
    if (!dst || !src) return ZNNI_ERR_NULL;
    if (bytes == 0 || (bytes & 15u)) return ZNNI_ERR_SHAPE;
    if (((uintptr_t)dst | (uintptr_t)src) & 15u) return ZNNI_ERR_ALIGN;
    const size_t n16 = bytes / 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 0x7fffffffull) blocks = 0x7fffffffull;     // beyond 8 TiB the kernel's loop takes over
    k_copy_probe<<<dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream>>>((float4*)dst, (const float4*)src, n16);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    return ZNNI_OK;
}

}  // extern "C"
