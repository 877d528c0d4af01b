// passes_tiles.hip -- z and y transforms of layers whose (y, z) planes are cut into overlapping tiles.
//
// A valid convolution may be computed tile by tile: V outputs along an axis need V + k - 1 inputs, so outputs are cut into tiles
// along y and z, and every tile goes through transforms of its own length N >= V + k - 1 (overlap-save).  x is not transformed.
// What that buys, against the separate z and y passes over whole planes (Section III-B/C):
//  * a tile's plane fits LDS, so z and y are one kernel a side and the tensors between them are gone: 8 N^2 bytes are written or
//    read per pair of tiles instead of three tensors of that size;
//  * kernel transforms are those of a tile, shared by all tiles: 48 -> 48 images of 320^3, 5^3 kernels 0.1 GB instead of 4.75.
// Against it stand the outputs that tiles share their inputs for: (N / V)^2 more of everything.  With the products
// in mac_quads.hip, whole layers: 48 -> 48 of 320^3, 5^3 15.7 -> 12.4 ms; 40 -> 40 of 128^3, 3^3 0.840 -> 0.616; 37 -> 45 of 93 x 110 x
// 131, 3 x 4 x 5 0.669 -> 0.490.  Since transforms are shorter, the results are 0.86 times as far from 64 bits on average, 0.64 to 1.08
// over 60 layers whose whole planes were multiplied on split halves as well; 0.74, 0.44 to 0.97 over 130 (0.98 with values spread over
// 2^12) that were transformed along x and multiplied in fp32: halves there too now, in closer sums.
//
// Two tiles of a plane ride as the real and the imaginary part of one complex plane, all the way: the products with the kernel
// transforms are linear, so nothing is taken apart in between, and both transforms are plain complex ones (a real transform of
// one tile needs an untangling on either side, and every pass through LDS has to know about it).  The spectra are whole complex
// planes [oz < N][oy < N] of half as many images, with as many products; pencils of the second half meet the conjugate kernel
// transforms of the first (mac_quads.hip).  The two tiles belong to one image and one x, so that no value meets another input's, or
// another x's, that it did not meet in the transforms of the whole plane.
//
// One workgroup takes four neighbouring x of one pair, one after the other, and holds their spectra in registers, so that 32
// bytes of a pencil's row are stored together (blocks of four x, as in passes_fused.hip).  Threads lie along lines: z while y is
// transformed, oy while z is, so that global loads and stores run along z, LDS is read and written with few bank conflicts (odd
// pitch: none at 32 and from 48 on, a fifth of the LDS cycles where a wave's lanes lie along more than one line), and up to 64 lines all twiddles of a wave are one, read as scalars.  Every step of a transform reads and writes the
// same LDS places, thread for thread, so that there are four barriers a plane (k_fwd_zy has nine).  Bound by memory: N = 36
// 5.5 TB/s (a copy reaches 6.2), 56 and 64 5.4; at 84 (one workgroup of sixteen waves per CU) 4.4.  Lengths whose workgroups do not
// fill the SIMDs evenly (60: ten waves) fall to 3.6 and are not offered.
#include "two_step.h"
#include <algorithm>
#include "mac_xd.h"

namespace znni {

struct TileArgs {
    const float* in;
    float* out;
    float2* X;             // X2 or Yd: [tile pair][image][oz][x / 4][oy][x % 4]
    const float2* tw;      // [N]
    const float* col;      // forward: powers of two of the f input images (mac_xd.hip)
    const float* bias;
    int f, relu;           // images (f or f') of an input
    int nx, ny, nz;        // the whole images (forward: input, inverse: output)
    int ntz, ntiles;       // tiles along z and altogether
    int Vy, Vz, Ey, Ez;    // outputs and rows of a tile
    int noy, noz;          // outputs of the whole image
    int ky, kz;
    int pairs, p0;         // tile pairs of this launch and the first of them
    int groups;            // S * f * blocks of four x
    int nxb;
};

// R1 <= R2.  A transform along an axis is a step of N / R threads a line and R values each, and the other way round; the outer
// steps, next to global memory, are those of R1 values by R2 threads.
template <int R1_, int R2_> struct Tile {
    static constexpr int R1 = R1_, R2 = R2_, N = R1 * R2, P = N | 1;
    static constexpr bool UNI = N > 48 && N <= 64;       // a wave per transform unit, lanes along lines
    static constexpr int LW = UNI ? 64 : N;
    static constexpr int NTH = (LW * R2 + 63) / 64 * 64;
    static constexpr int REGION = (N * P + 1) & ~1;
    static constexpr size_t LDS = sizeof(float2) * (size_t)(REGION + (UNI ? 0 : N));
};

typedef const __attribute__((address_space(4))) float2* ScalarTw;

template <typename TL, int R>
__device__ __forceinline__ void tile_twiddle(float2 (&v)[R], int j, const float2* twg, const float2* tws)
{
#pragma unroll
    for (int q = 1; q < R; ++q) {
        float2 w;
        if constexpr (TL::UNI) {
            const ScalarTw p = (ScalarTw)twg + j * q;
            w = make_float2(p->x, p->y);
        } else w = tws[j * q];
        v[q] = cmul(v[q], w);
    }
}

// First output (and input) row of a tile along y and z.  Tiles at the end are moved back so that all have one size; the outputs
// below ylo and zlo are the tile's before.
struct TilePos { int y, z, ylo, zlo; };
__device__ __forceinline__ TilePos tile_pos(const TileArgs& a, int t)
{
    const int ty = t / a.ntz, tz = t - ty * a.ntz;
    TilePos r;
    r.y = min(ty * a.Vy, a.noy - a.Vy);
    r.z = min(tz * a.Vz, a.noz - a.Vz);
    r.ylo = ty * a.Vy - r.y;
    r.zlo = tz * a.Vz - r.z;
    return r;
}

// The pairs of a block of four x are neighbours on one XCD: they share the rows they overlap in.
template <int R1, int R2>
__global__ __launch_bounds__((Tile<R1, R2>::NTH)) __attribute__((amdgpu_waves_per_eu(4)))
void k_fwd_tiles(TileArgs a)
{
    using TL = Tile<R1, R2>;
    constexpr int N = TL::N, P = TL::P;
    extern __shared__ float2 lds[];
    float2* const R = lds;
    float2* const tws = lds + TL::REGION;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int gq = slot / a.pairs, p = slot - gq * a.pairs, grp = gq * 8 + xcd;
    if (grp >= a.groups) return;
    const int img = grp / a.nxb, xb = grp - img * a.nxb;
    const int t0 = 2 * (a.p0 + p);
    const TilePos ta = tile_pos(a, t0), tb = tile_pos(a, min(t0 + 1, a.ntiles - 1));
    const int t = threadIdx.x;
    int line = t % TL::LW, unit = t / TL::LW;
    if constexpr (TL::UNI) unit = __builtin_amdgcn_readfirstlane(unit);
    else for (int q = t; q < N; q += TL::NTH) tws[q] = a.tw[q];
    const bool all = line < N && unit < R2, some = line < N && unit < R1;
    const int left = a.nx - 4 * xb;
    const size_t pl = (size_t)a.ny * a.nz;
    const float* const in0 = a.in + ((size_t)img * a.nx + 4 * xb) * pl;
    const float* const ia = in0 + (size_t)ta.y * a.nz + ta.z;
    const float* const ib = in0 + (size_t)tb.y * a.nz + tb.z;
    const float ps = a.col ? a.col[img % a.f] : 1.f;
    const int zl = min(line, a.Ez - 1);

    // (rows and columns beyond a tile repeat its last ones: they reach no output that is kept)
    float ra[R1], rb[R1];
    auto request = [&](int h) {
        const size_t o = (size_t)min(h, left - 1) * pl;
#pragma unroll
        for (int m = 0; m < R1; ++m) {
            const int y = min(unit + R2 * m, a.Ey - 1);
            const int off = y * a.nz;
            if constexpr (TL::UNI) {
                ra[m] = (ia + o + off)[zl];
                rb[m] = (ib + o + off)[zl];
            } else {
                ra[m] = (ia + o)[off + zl];
                rb[m] = (ib + o)[off + zl];
            }
        }
    };
    if (all) request(0);
    struct alignas(16) Run { float2 v[4]; } keep[R1];
    if constexpr (!TL::UNI) __syncthreads();
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float2 v[R1], u[R2];
        // along y, a thread per (z, unit): values unit + R2 m
        if (all) {
#pragma unroll
            for (int m = 0; m < R1; ++m) v[m] = make_float2(ra[m] * ps, rb[m] * ps);
            Dft<R1>::run(v);
            tile_twiddle<TL>(v, unit, a.tw, tws);
        }
        if (h) __syncthreads();
        if (all) {
#pragma unroll
            for (int q = 0; q < R1; ++q) R[(q + R1 * unit) * P + line] = v[q];
        }
        __syncthreads();
        if (h < 3 && all) request(h + 1);     // (in flight while this plane is transformed)
        if (some) {
#pragma unroll
            for (int j = 0; j < R2; ++j) u[j] = R[(unit + R1 * j) * P + line];
            Dft<R2>::run(u);
#pragma unroll
            for (int r = 0; r < R2; ++r) R[(unit + R1 * r) * P + line] = u[r];
        }
        __syncthreads();
        // along z, a thread per (oy, unit)
        if (some) {
#pragma unroll
            for (int m = 0; m < R2; ++m) u[m] = R[line * P + unit + R1 * m];
            Dft<R2>::run(u);
            tile_twiddle<TL>(u, unit, a.tw, tws);
#pragma unroll
            for (int q = 0; q < R2; ++q) R[line * P + unit + R1 * q] = u[q];
        }
        __syncthreads();
        if (all) {
#pragma unroll
            for (int j = 0; j < R1; ++j) v[j] = R[line * P + unit * R1 + j];
            Dft<R1>::run(v);
#pragma unroll
            for (int r = 0; r < R1; ++r) keep[r].v[h] = v[r];
        }
    }
    if (all) {
        const int s = img / a.f, i = img - s * a.f;
        Run* dst = reinterpret_cast<Run*>(a.X) + (((size_t)(s * a.pairs + p) * a.f + i) * N * a.nxb + xb) * N + line;
#pragma unroll
        for (int r = 0; r < R1; ++r) dst[(size_t)(unit + R2 * r) * a.nxb * N] = keep[r];
    }
}

// The mirror image: conj . forward . conj along z, then along y; the real part belongs to the first tile, minus the imaginary part
// to the second.
template <int R1, int R2>
__global__ __launch_bounds__((Tile<R1, R2>::NTH)) __attribute__((amdgpu_waves_per_eu(4)))
void k_inv_tiles(TileArgs a)
{
    using TL = Tile<R1, R2>;
    constexpr int N = TL::N, P = TL::P;
    extern __shared__ float2 lds[];
    float2* const R = lds;
    float2* const tws = lds + TL::REGION;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int gq = slot / a.pairs, p = slot - gq * a.pairs, grp = gq * 8 + xcd;
    if (grp >= a.groups) return;
    const int img = grp / a.nxb, xb = grp - img * a.nxb;
    const int t = threadIdx.x;
    int line = t % TL::LW, unit = t / TL::LW;
    if constexpr (TL::UNI) unit = __builtin_amdgcn_readfirstlane(unit);
    const bool all = line < N && unit < R2, some = line < N && unit < R1;
    struct alignas(16) Run { float2 v[4]; } raw[R1];
    const int s = img / a.f, i = img - s * a.f;
    if (all) {
        const Run* src = reinterpret_cast<const Run*>(a.X) + (((size_t)(s * a.pairs + p) * a.f + i) * N * a.nxb + xb) * N + line;
#pragma unroll
        for (int m = 0; m < R1; ++m) raw[m] = src[(size_t)(unit + R2 * m) * a.nxb * N];
    }
    if constexpr (!TL::UNI) {
        for (int q = t; q < N; q += TL::NTH) tws[q] = a.tw[q];
        __syncthreads();
    }
    const int t0 = 2 * (a.p0 + p);
    const bool two = t0 + 1 < a.ntiles;
    const TilePos ta = tile_pos(a, t0), tb = tile_pos(a, two ? t0 + 1 : t0);
    const int left = a.nx - 4 * xb;
    const size_t pl = (size_t)a.ny * a.nz;
    float* const out0 = a.out + ((size_t)img * a.nx + 4 * xb) * pl;
    float* const oa = out0 + (size_t)ta.y * a.nz + ta.z;
    float* const ob = out0 + (size_t)tb.y * a.nz + tb.z;
    const float bj = a.bias ? a.bias[i] : 0.f;
    const int zo = line - (a.kz - 1);
    const bool za = zo >= ta.zlo && zo < a.Vz, zb = two && zo >= tb.zlo && zo < a.Vz;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        if (h >= left) break;
        float2 v[R1], u[R2];
        if (all) {
#pragma unroll
            for (int m = 0; m < R1; ++m) v[m] = cconj(raw[m].v[h]);
            Dft<R1>::run(v);
            tile_twiddle<TL>(v, unit, a.tw, tws);
        }
        if (h) __syncthreads();
        if (all) {
#pragma unroll
            for (int q = 0; q < R1; ++q) R[line * P + q + R1 * unit] = v[q];
        }
        __syncthreads();
        if (some) {
#pragma unroll
            for (int j = 0; j < R2; ++j) u[j] = R[line * P + unit + R1 * j];
            Dft<R2>::run(u);
#pragma unroll
            for (int r = 0; r < R2; ++r) R[line * P + unit + R1 * r] = u[r];
        }
        __syncthreads();
        if (some) {
#pragma unroll
            for (int m = 0; m < R2; ++m) u[m] = R[(unit + R1 * m) * P + line];
            Dft<R2>::run(u);
            tile_twiddle<TL>(u, unit, a.tw, tws);
#pragma unroll
            for (int q = 0; q < R2; ++q) R[(unit + R1 * q) * P + line] = u[q];
        }
        __syncthreads();
        if (all) {
#pragma unroll
            for (int j = 0; j < R1; ++j) v[j] = R[(unit * R1 + j) * P + line];
            Dft<R1>::run(v);
#pragma unroll
            for (int r = 0; r < R1; ++r) {
                const int yo = unit + R2 * r - (a.ky - 1);
                const size_t o = h * pl;
                float va = v[r].x + bj, vb = bj - v[r].y;
                if (a.relu) { va = fmaxf(va, 0.f); vb = fmaxf(vb, 0.f); }
                if constexpr (TL::UNI) {
                    if (yo < a.Vy) {
                        if (yo >= ta.ylo && za) (oa + o + yo * a.nz)[zo] = va;
                        if (yo >= tb.ylo && zb) (ob + o + yo * a.nz)[zo] = vb;
                    }
                } else {
                    if (za && yo >= ta.ylo && yo < a.Vy) (oa + o)[yo * a.nz + zo] = va;
                    if (zb && yo >= tb.ylo && yo < a.Vy) (ob + o)[yo * a.nz + zo] = vb;
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------- host side
static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

bool tiles_plan(const LayerPlan& whole, int N, void* base, size_t room, bool chunks, LayerPlan* out)
{
    LayerPlan L = whole;
    Dims& d = L.d;
    auto& c = L.cut;
    if (N < 1 || d.ky > N || d.kz > N) return false;
    c.S = whole.S; c.ny = d.ny; c.nz = d.nz; c.noy = d.noy; c.noz = d.noz;
    const int my = N - d.ky + 1, mz = N - d.kz + 1;
    c.nty = (d.noy + my - 1) / my; c.ntz = (d.noz + mz - 1) / mz;
    d.noy = (c.noy + c.nty - 1) / c.nty; d.noz = (c.noz + c.ntz - 1) / c.ntz;
    d.ny = d.noy + d.ky - 1; d.nz = d.noz + d.kz - 1;
    d.Ny = d.Nz = N;
    d.zc = N / 2 + 1;
    c.pairs = (c.nty * c.ntz + 1) / 2;
    L.tiles = L.planes = L.xdirect = true;
    L.xblock = false;
    const size_t e = sizeof(float2), per = (size_t)d.kx * L.fp * L.Mp * e;
    uintptr_t p = (uintptr_t)base;
    auto take = [&](size_t bytes) { const uintptr_t q = p; p += up256(bytes); return (float2*)q; };
    L.twx = take(d.Nx * e); L.twy = take(N * e); L.twz = take(N * e);
    L.A1 = take(d.zc * d.ky * per);
    L.A = take((size_t)d.zc * N * per);
    L.rs = (float*)take(split_scale_floats(L) * sizeof(float));
    L.oz0 = 0; L.ozn = d.zc;
    const size_t fixed = p - (uintptr_t)base + 512;
    const size_t xp = (size_t)N * N * ((d.nx + 3) / 4) * 4 * e * L.f, yp = (size_t)N * N * ((d.nox + 3) / 4) * 4 * e * L.fo;
    if (room < fixed) return false;
    const long long fit = (long long)((room - fixed) / (xp + yp));
    c.s0 = c.p0 = 0; c.sn = c.S; c.pn = c.pairs;
    if (fit < (long long)c.S * c.pairs) {
        if (!chunks || fit < 1) return false;
        if (fit >= c.pairs) c.sn = (int)(fit / c.pairs);
        else {
            c.sn = 1;
            const int parts = (int)((c.pairs + fit - 1) / fit);
            c.pn = (c.pairs + parts - 1) / parts;
        }
    }
    L.S = c.sn * c.pn; L.nimg = L.S * L.f; L.nimgo = L.S * L.fo;
    L.buf1 = take(xp * L.S);
    L.Yt = L.buf0 = take(yp * L.S);
    *out = L;
    return true;
}

// The lengths that are instantiated, and what the transform kernels of each were measured to take (1500 random layers): a launch
// and the tail of its last workgroups, and bytes per second behind that.
struct TileLength { int N; float fwd_us, fwd_tbs, inv_us, inv_tbs; };
static const TileLength kTileLengths[] = {
    {24, 8.4f, 5.78f, 8.3f, 5.30f},  {28, 9.2f, 6.14f, 8.6f, 5.23f},  {32, 9.3f, 6.32f, 8.2f, 5.50f},  {36, 9.3f, 6.18f, 8.7f, 5.26f},
    {40, 8.9f, 5.36f, 8.2f, 4.59f},  {42, 8.8f, 5.30f, 8.2f, 4.49f},  {48, 10.5f, 5.28f, 9.6f, 4.72f}, {56, 11.4f, 5.77f, 9.6f, 4.96f},
    {64, 11.7f, 5.78f, 9.4f, 5.11f}, {72, 12.9f, 4.46f, 9.7f, 3.76f}, {84, 11.5f, 4.29f, 10.1f, 3.91f}};

// Waves of a multiply-accumulate, what they multiply (column and row tiles times matrix steps) and stage (chunks of images).
struct MacWaves { double waves, products, chunks; };
static MacWaves mac_waves(const LayerPlan& L, int CT, double pencils)
{
    const double w = pencils * L.mac_nmblk * ((L.d.nox + 16 * CT - 1) / (16 * CT));
    return MacWaves{w, w * ((L.d.kx * (L.fp >> 2) + 3) / 4) * L.mac_RTW * CT, w * ((L.f + 15) / 16)};
}

// Estimated times, without the kernel transforms (which a call may keep) and with them.
struct Seconds { double kept, all; };
static Seconds tiles_estimate(const LayerPlan& L)
{
    const Dims& d = L.d;
    const auto& c = L.cut;
    const TileLength* t = kTileLengths;
    while (t->N != d.Ny) ++t;
    const double E = (double)c.S * c.pairs, plane = 8.0 * d.Ny * d.Nz, tiles = (double)c.S * c.nty * c.ntz;
    const double xb = (d.nx + 3) / 4 * 4 * plane * E * L.f, yb = (d.nox + 3) / 4 * 4 * plane * E * L.fo;
    const double per = 8.0 * d.zc * d.kx * L.fp * (double)L.Mp, bank = per * d.Ny, a1 = per * d.ky;
    const MacWaves m = mac_waves(L, quads_strip(L), E * d.Nz * ((d.Ny + 3) & ~3));
    const double turns = (double)((c.S + c.sn - 1) / c.sn) * ((c.pairs + c.pn - 1) / c.pn);
    double us = turns * (t->fwd_us + t->inv_us + 5.7);
    us += (4.0 * tiles * L.f * d.nx * d.ny * (double)d.nz + xb) / t->fwd_tbs * 1e-6;
    us += (4.0 * tiles * L.fo * d.nox * d.noy * (double)d.noz + yb) / t->inv_tbs * 1e-6;
    static const float product[] = {3.3e-5f, 4.8e-5f, 5.3e-5f, 5.9e-5f, 6.4e-5f};        // by row tiles
    us += product[L.mac_RTW - 1] * m.products + 2.9e-4 * m.chunks + 7e-4 * m.waves + (xb + yb + bank) / 5.6e6;
    return Seconds{us * 1e-6, (us + 11 + bank / 9.0e6 + a1 / 0.80e6) * 1e-6};
}
double tiles_seconds(const LayerPlan& L) { return tiles_estimate(L).all; }

// The whole planes' route, likewise (1015 random layers whose x axis is not transformed: 1.04 of the time measured, a tenth of them
// below 0.91 and above 1.22 of it; tiles 1.01, 0.89 and 1.12).
static Seconds whole_estimate(const LayerPlan& L)
{
    if (!L.xdirect) { const double s = 1.15 * route_seconds(L); return Seconds{s, s}; }
    const Dims& d = L.d;
    double hb[ZNNI_NUM_STAGES], fl[ZNNI_NUM_STAGES];
    plan_work(L, 0, hb, fl);
    const double per = 8.0 * d.zc * d.kx * L.fp * (double)L.Mp, bank = per * d.Ny, a1 = per * d.ky;
    const int tiles = (d.nox + 15) / 16;
    const MacWaves m = mac_waves(L, std::min(tiles, L.mac_RTW < 4 ? 4 : 2), (double)L.S * d.Ny * d.zc);
    double us = 32 + hb[ZNNI_STAGE_FWD_Z] / 4.9e6 + hb[ZNNI_STAGE_FWD_Y] / 5.35e6 + hb[ZNNI_STAGE_INV_Y] / 5.8e6 + hb[ZNNI_STAGE_INV_Z] / 5.5e6;
    // (stepwise sums or not: launch_xd_cols in mac_xd.hip)
    us += (mac_xb_available(L) || mac_batch_preferred(L) ? 4.3e-5 : 3.55e-5) * m.products + 3.7e-4 * m.chunks + 2.8e-4 * m.waves + hb[ZNNI_STAGE_MAC] / 6.6e6;
    return Seconds{us * 1e-6, (us + 11.6 + bank / 6.6e6 + a1 / 1.15e6) * 1e-6};
}

// The length whose estimate is the lowest, if that is below the whole planes' by a twelfth, with kernel transforms and without.
// Over 1015 random layers of 2 to 100 images of 24 to 320 an edge, 834 of which go in tiles: 1.29 times as fast on average (1.26 with
// kept kernel transforms), two more than 3 % behind whole planes, the worst 6 % (1 x 3 -> 6 of 341 x 227 x 155, 3 x 6 x 9: few images
// leave chunks of sixteen empty); the pick is 0.5 % off the best length.  Layers that already go four planes at a time stay there
// (they have two kernels around the product as well, and lengths that fit), and so do layers below 60 us: launches.  With many
// products per value moved, more products cost more than fewer passes save (80 -> 80 of 128^3, 7^3: passes 1030 -> 700 us,
// multiply-accumulate 1020 -> 1560).
int pick_tiles(const LayerPlan& whole, size_t room, bool chunks)
{
    if (whole.generic_passes || whole.planes || !mac_xd_available(whole)) return 0;
    const Seconds w = whole_estimate(whole);
    if (w.kept < 60e-6) return 0;
    int N = 0;
    double best = 0.92 * w.all;
    LayerPlan T;
    for (const TileLength& t : kTileLengths)
        if (tiles_plan(whole, t.N, nullptr, room, chunks, &T)) {
            const Seconds s = tiles_estimate(T);
            if (s.all < best && s.kept < 0.92 * w.kept) { best = s.all; N = t.N; }
        }
    return N;
}

static void tile_args(const LayerPlan& L, TileArgs* a)
{
    const Dims& d = L.d;
    const auto& c = L.cut;
    a->tw = L.twy; a->ny = c.ny; a->nz = c.nz; a->ntz = c.ntz; a->ntiles = c.nty * c.ntz;
    a->Vy = d.noy; a->Vz = d.noz; a->Ey = d.ny; a->Ez = d.nz; a->noy = c.noy; a->noz = c.noz; a->ky = d.ky; a->kz = d.kz;
    a->pairs = c.pn; a->p0 = c.p0;
    a->col = nullptr; a->bias = nullptr; a->relu = 0; a->in = nullptr; a->out = nullptr;
}

template <int R1, int R2, bool FWD>
static znni_status launch_tiles(const TileArgs& a, hipStream_t st)
{
    using TL = Tile<R1, R2>;
    void (*kernel)(TileArgs) = FWD ? k_fwd_tiles<R1, R2> : k_inv_tiles<R1, R2>;
    const long long blocks = (long long)((a.groups + 7) / 8) * 8 * a.pairs;
    if (blocks > 0x7fffffffll) return ZNNI_ERR_SHAPE;
    if (TL::LDS > 48 * 1024 && hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TL::LDS) != hipSuccess)
        return ZNNI_ERR_HIP;
    kernel<<<dim3((unsigned)blocks), dim3(TL::NTH), TL::LDS, st>>>(a);
    return hipGetLastError() == hipSuccess ? ZNNI_OK : ZNNI_ERR_HIP;
}
template <bool FWD>
static znni_status launch_tiles(const TileArgs& a, int N, hipStream_t st)
{
    switch (N) {
        case 24: return launch_tiles<4, 6, FWD>(a, st);
        case 28: return launch_tiles<4, 7, FWD>(a, st);
        case 32: return launch_tiles<4, 8, FWD>(a, st);
        case 36: return launch_tiles<6, 6, FWD>(a, st);
        case 40: return launch_tiles<5, 8, FWD>(a, st);
        case 42: return launch_tiles<6, 7, FWD>(a, st);
        case 48: return launch_tiles<6, 8, FWD>(a, st);
        case 56: return launch_tiles<7, 8, FWD>(a, st);
        case 64: return launch_tiles<8, 8, FWD>(a, st);
        case 72: return launch_tiles<8, 9, FWD>(a, st);
        case 84: return launch_tiles<7, 12, FWD>(a, st);
    }
    return ZNNI_ERR_UNSUPPORTED_SIZE;
}

znni_status launch_fwd_tiles(const LayerPlan& L, const float* in, hipStream_t st)
{
    TileArgs a;
    tile_args(L, &a);
    const auto& c = L.cut;
    a.f = L.f; a.nx = L.d.nx; a.nxb = (a.nx + 3) / 4; a.groups = c.sn * L.f * a.nxb;
    a.in = in + (size_t)c.s0 * L.f * a.nx * c.ny * c.nz; a.X = L.buf1; a.col = split_scales(L).col;
    return launch_tiles<true>(a, L.d.Ny, st);
}

znni_status launch_inv_tiles(const LayerPlan& L, const float* bias, float* out, unsigned flags, hipStream_t st)
{
    TileArgs a;
    tile_args(L, &a);
    const auto& c = L.cut;
    a.f = L.fo; a.nx = L.d.nox; a.nxb = (a.nx + 3) / 4; a.groups = c.sn * L.fo * a.nxb;
    a.ny = c.noy; a.nz = c.noz;
    a.out = out + (size_t)c.s0 * L.fo * a.nx * c.noy * c.noz; a.X = L.Yt; a.bias = bias; a.relu = (flags & ZNNI_RELU) ? 1 : 0;
    return launch_tiles<false>(a, L.d.Ny, st);
}

}  // namespace znni
