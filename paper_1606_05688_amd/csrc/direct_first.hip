// direct_first.hip -- direct convolution of layers of 13 to 64 taps over all input images: a network's first layers.
//
// The same contraction as direct.hip's over (input image, tap), with the shifted image values read from a tile in LDS, for layers
// with so few products per output that the result's writing should be the bound.  There, the fp32 matrix instructions take as long as
// the stores (one image to 48, 128^3, 3^3: 67 us at their rate, next to 62 us of stores), so every value is three halves, which hold
// all 24 bits of it: one or two steps of 32 taps on v_mfma_f32_16x16x32_f16, the six partial products that reach the result
// (error against 64 bits 0.51 of the fp32 kernel's on average over 188 layers, 0.69 at most).  A tile has one power of two, an output
// image's kernels another: exact for values down to 2^-37 of the largest.  Where magnitudes lie further apart than that, or are not
// finite, the tile is multiplied in fp32, from the same registers (that layer 119 us, 124 by the fp32 kernel; over those layers 1.05
// times as fast as by that kernel, 0.69 at worst).  Two halves instead of three are 6 % faster here (10 % over those layers), but
// drop a bit of every fourth value, and more below 2^-17 of the largest.
//
// A workgroup keeps its kernels' operands in registers and walks over tiles of 256 outputs of an image (128, 64 or 32 columns, the
// others rows): values of the next tile are requested before this one is multiplied.  What decided, on that layer (124 us before):
// * all workgroups' tiles of a turn lie next to each other, an XCD's in one run.  A run of tiles a workgroup: 123 us, as its stores
//   went to as many places as there are workgroups times images; one tile a workgroup: 253 us, the kernels' operands made each time.
// * stores of 256-byte runs (through LDS), 16 bytes a lane, without a branch: the wait for the next tile's values then does not
//   wait for them.  64-byte runs straight from the accumulators: 121 us.  Nontemporal stores: 214 us (rows end inside lines).
// Now 101 us, 3.9 TB/s of the 6.2 that a copy reaches; what is left is waiting at the two barriers of a turn, and LDS: eight bytes a
// staged value.  (The figures above are from two halves a value, of 95 us.)
#include <math.h>

#include <algorithm>

#include "direct_split.h"
#include "split.h"

namespace znni {

typedef float floatx4_f __attribute__((ext_vector_type(4)));

constexpr int FIRST_NQ = 13;                      // staged values of a thread, at most
// Workgroups a compute unit: one row tile three (two 4 to 14 % slower over 319 layers), two to five row tiles two (three 3 to 17 % slower).
constexpr int first_resident(int RTW) { return RTW == 1 ? 3 : 2; }
constexpr int first_slots(int RTW) { return 256 * first_resident(RTW); }
constexpr int FIRST_SPAN = 37;                    // three halves are exact for values down to 2^-37 of the largest
constexpr int FIRST_P = 68;                       // pitch of a wave's rows on their way out: no bank conflicts either way
constexpr unsigned FIRST_NONE = 0xfffffff0u;     // an offset that the range check of loads and stores drops

struct FirstArgs {
    const float *in, *w, *bias;
    float* out;
    Dims d;
    int f, fo, K, taps;          // K: taps of all input images
    int TZ, TY;                  // columns (32, 64 or 128) and rows of a tile: 256 outputs of an image
    int TYI, TZI, tilevol, total;
    int nty, ntz, tiles;         // tiles of an input's image along y and z, of all inputs
    FastDiv by_vol, by_tz, by_ty, by_taps, by_kz, by_ky, by_ntz, by_nty, by_nox;
    int relu;
};

// NQ: staged values per thread; ST: steps of 32 taps; RTW: row tiles of 16 output images.  Bound by the result's writing (where many
// images are written) or by a turn's latency.
template <int RTW, int ST, int NQ>
__global__ __launch_bounds__(256, first_resident(RTW)) void k_direct_first(FirstArgs a)
{
    extern __shared__ unsigned lds_u[];
    uint2* const th = reinterpret_cast<uint2*>(lds_u);            // staged values: three halves each, or fp32
    int* const delta = reinterpret_cast<int*>(lds_u + 2 * ((a.total + 1) & ~1));   // [64] offset of a tap inside the tile
    unsigned* const red = reinterpret_cast<unsigned*>(delta + 64);             // [turn][largest, smallest]
    float* const out = reinterpret_cast<float*>(red + 8);                      // [wave][16][FIRST_P]
    const Dims& d = a.d;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, l16 = lane & 15, kk = lane >> 4;
    const int rt0 = blockIdx.y * RTW;
    const int nb = gridDim.x, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int chunk = xcd * (nb >> 3) + min(xcd, nb & 7) + slot;  // (neighbours in memory on one XCD)
    const int tile0 = chunk;
    if (tile0 >= a.tiles) return;

    // ---- where this thread's values of a tile lie, from the tile's first
    const unsigned nyz = (unsigned)d.ny * d.nz, nvox = nyz * d.nx;
    unsigned lo[NQ];
    float raw[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const unsigned e = t + 256 * q, i = a.by_vol.div(e), v = e - i * a.tilevol, y = a.by_tz.div(v), lz = v - y * a.TZI;
        const unsigned lx = a.by_ty.div(y), ly = y - lx * a.TYI;
        lo[q] = e < (unsigned)a.total ? 4u * (i * nvox + lx * nyz + ly * d.nz + lz) : FIRST_NONE;
        raw[q] = 0.f;
    }
    int s, x0, y0, z0;
    auto place = [&](int tile) {
        const int q = (int)a.by_ntz.div(tile), x = (int)a.by_nty.div(q);
        s = (int)a.by_nox.div(x); x0 = x - s * d.nox; y0 = (q - x * a.nty) * a.TY; z0 = (tile - q * a.ntz) * a.TZ;
    };
    // (rows and columns past an image's end read what follows them in this input's images, zeros past the last: they enter
    // results that are not stored, and the choice of the scale)
    auto request = [&](int tile) {
        place(tile);
        const size_t at = (size_t)((x0 * d.ny + y0) * d.nz + z0), all = (size_t)a.f * nvox;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.in) + s * all + at, 0, (int)(unsigned)(4 * (all - at)), 0x00020000);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (256 * q < a.total) raw[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lo[q], 0, 0));
    };
    request(tile0);

    // ---- kernels: operands of all steps in registers, a power of two per output image
    half8 wh[ST][RTW], wm[ST][RTW], wl[ST][RTW];
    int we[RTW];
    float bj[RTW];
    bool wide = false;
    {
        float v[RTW][ST][8];
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            const int j = min((rt0 + r) * 16 + l16, a.fo - 1);
            bj[r] = a.bias ? a.bias[j] : 0.f;
#pragma unroll
            for (int st = 0; st < ST; ++st)
#pragma unroll
                for (int u = 0; u < 8; ++u) v[r][st][u] = a.w[j * a.K + min(st * 32 + u * 4 + kk, a.K - 1)];
        }
        // (all requested before the first is looked at: a load behind a branch each took a round trip to memory each)
#pragma unroll
        for (int r = 0; r < RTW; ++r)
#pragma unroll
            for (int st = 0; st < ST; ++st)
#pragma unroll
                for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(v[r][st][u]));
        if (t < 64) {
            const int k = t, i = (int)a.by_taps.div(k), q = k - i * a.taps, y = (int)a.by_kz.div(q), c = q - y * d.kz, x = (int)a.by_ky.div(y), b = y - x * d.ky;
            delta[t] = k < a.K ? i * a.tilevol + ((d.kx - 1 - x) * a.TYI + (d.ky - 1 - b)) * a.TZI + (d.kz - 1 - c) : 0;
        }
        if (t < 6) red[t] = t & 1 ? ~0u : 0u;
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            unsigned m = 0, mn = ~0u;
#pragma unroll
            for (int st = 0; st < ST; ++st)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    v[r][st][u] = st * 32 + u * 4 + kk < a.K ? v[r][st][u] : 0.f;
                    const float ax = fabsf(v[r][st][u]);
                    m = max(m, __float_as_uint(ax));              // (NaNs are the largest)
                    mn = min(mn, small_code(ax));
                }
#pragma unroll
            for (int o = 16; o < 64; o <<= 1) {
                m = max(m, (unsigned)__shfl_xor((int)m, o));
                mn = min(mn, (unsigned)__shfl_xor((int)mn, o));
            }
            const bool bad = m >= 0x7f800000u || split_too_wide(m, mn, FIRST_SPAN);
            wide |= __ballot(bad) != 0;
            we[r] = split_exp(bad ? 0.f : __uint_as_float(m));
        }
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            const float sc = pow2f(we[r]);
#pragma unroll
            for (int st = 0; st < ST; ++st) {
                if (wide) {                                       // fp32 as it is, in the place of the first two halves
                    uintx4 a0, a1;
#pragma unroll
                    for (int u = 0; u < 4; ++u) { a0[u] = __float_as_uint(v[r][st][u]); a1[u] = __float_as_uint(v[r][st][4 + u]); }
                    wh[st][r] = __builtin_bit_cast(half8, a0); wm[st][r] = __builtin_bit_cast(half8, a1);
                } else {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        _Float16 h, c, l;
                        split3(v[r][st][u], sc, h, c, l);
                        wh[st][r][u] = h; wm[st][r][u] = c; wl[st][r][u] = l;
                    }
                }
            }
        }
    }
    __syncthreads();
    int dl[ST][8];
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int u = 0; u < 8; ++u) dl[st][u] = delta[st * 32 + u * 4 + kk];

    float* const mine = out + wave * 16 * FIRST_P;
    const unsigned ovox = (unsigned)d.nox * d.noy * d.noz;
    // a wave: 64 columns of one output row, or 32 of two
    const bool two = a.TZ == 32;
    const int row = two ? 2 * wave : a.TZ == 64 ? wave : wave >> 1, zb = a.TZ == 128 ? (wave & 1) * 64 : 0;
    const uint2* const base = th + row * a.TZI + zb + l16;
    int next = two ? a.TZI : 32;                                  // ... to the other two column tiles
    const int half = two && l16 >= 8, zl = 4 * l16 - 32 * half;             // row and first column of what this lane stores
    for (int tile = tile0, turn = 0; tile < a.tiles; tile += nb, turn = turn == 2 ? 0 : turn + 1) {
        unsigned m = 0, mn = ~0u;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const float ax = fabsf(raw[q]);
            m = max(m, __float_as_uint(ax));
            mn = min(mn, small_code(ax));
        }
        {
            const unsigned wm = wave_max(__uint_as_float(m)), wn = wave_min(mn);
            if (lane == 0) { atomicMax(red + 2 * turn, wm); atomicMin(red + 2 * turn + 1, wn); }
        }
        __syncthreads();                                          // (also: all waves are through with the tile before)
        const unsigned most = __builtin_amdgcn_readfirstlane(red[2 * turn]), least = __builtin_amdgcn_readfirstlane(red[2 * turn + 1]);
        const bool exact = wide || most >= 0x7f800000u || split_too_wide(most, least, FIRST_SPAN);
        const int sx = exact ? 0 : split_exp(__uint_as_float(most));
        const float sc = pow2f(sx);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (256 * q >= a.total) continue;
            uint2 v = make_uint2(__float_as_uint(raw[q]), 0u);
            if (!exact) {
                _Float16 h, c, l;
                split3(raw[q], sc, h, c, l);
                v.x = (unsigned)__builtin_bit_cast(unsigned short, h) | (unsigned)__builtin_bit_cast(unsigned short, c) << 16;
                v.y = __builtin_bit_cast(unsigned short, l);
            }
            if (t + 256 * q < a.total) th[t + 256 * q] = v;
        }
        if (t < 2) red[2 * (turn == 0 ? 2 : turn - 1) + t] = t & 1 ? ~0u : 0u;
        __syncthreads();
        place(tile);
        const int Y = y0 + row, zn = Y + half < d.noy ? d.noz - (z0 + zb) : 0;   // columns of this lane's row to store (64 or more: all)
        float* const dst = a.out + (size_t)(s * a.fo + rt0 * 16) * ovox + ((size_t)x0 * d.noy + Y) * d.noz + z0 + zb;
        if (tile + nb < a.tiles) request(tile + nb);

        floatx4_f acc[RTW][4];
#pragma unroll
        for (int r = 0; r < RTW; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] = floatx4_f{0.f, 0.f, 0.f, 0.f};
        asm volatile("" : "+v"(next));                              // (their addresses are made again, not kept)
        const uint2* const base2 = base + next;
        if (!exact) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    uint2 p[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) p[u] = (c < 2 ? base : base2)[16 * (c & 1) + dl[st][u]];
                    uintx4 hh, mm, ll;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        hh[u] = __builtin_amdgcn_perm(p[2 * u + 1].x, p[2 * u].x, 0x05040100u);
                        mm[u] = __builtin_amdgcn_perm(p[2 * u + 1].x, p[2 * u].x, 0x07060302u);
                        ll[u] = __builtin_amdgcn_perm(p[2 * u + 1].y, p[2 * u].y, 0x05040100u);
                    }
                    const half8 xh = __builtin_bit_cast(half8, hh), xm = __builtin_bit_cast(half8, mm), xl = __builtin_bit_cast(half8, ll);
                    // the smallest products first, each group under its power of two
                    __builtin_amdgcn_s_setprio(1);                // (also keeps the operands of several steps out of the registers)
                    floatx4_f low[RTW];
#define ZNNI_FIRST(D, X, W, C)                  \
    _Pragma("unroll") for (int r = 0; r < RTW; ++r) D = __builtin_amdgcn_mfma_f32_16x16x32_f16(X, W[st][r], C, 0, 0, 0)
                    ZNNI_FIRST(low[r], xl, wh, (floatx4_f{0.f, 0.f, 0.f, 0.f}));
                    ZNNI_FIRST(low[r], xm, wm, low[r]);
                    ZNNI_FIRST(low[r], xh, wl, low[r]);
#pragma unroll
                    for (int r = 0; r < RTW; ++r) low[r] *= SPLIT3_STEP;
                    ZNNI_FIRST(low[r], xm, wh, low[r]);
                    ZNNI_FIRST(low[r], xh, wm, low[r]);
                    ZNNI_FIRST(acc[r][c], xh, wh, acc[r][c]);
#undef ZNNI_FIRST
                    __builtin_amdgcn_s_setprio(0);
#pragma unroll
                    for (int r = 0; r < RTW; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[r][c][e] = fmaf(low[r][e], SPLIT3_STEP, acc[r][c][e]);
                }
        } else {
            // fp32, with the operands where they are: a matrix step's four taps are the u-th of each lane group.  (Hidden from the compiler,
            // which would otherwise keep all kernel values in registers over the loop.)
            auto hide = [](half8& v) {
                uintx4 b = __builtin_bit_cast(uintx4, v);
                asm volatile("" : "+v"(b));
                v = __builtin_bit_cast(half8, b);
            };
#pragma unroll
            for (int st = 0; st < ST; ++st)
#pragma unroll
                for (int r = 0; r < RTW; ++r) { hide(wh[st][r]); hide(wm[st][r]); hide(wl[st][r]); }
#pragma unroll
            for (int st = 0; st < ST; ++st)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (st * 32 + u * 4 >= a.K) continue;
                    float x[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float xv = __uint_as_float((c < 2 ? base : base2)[16 * (c & 1) + dl[st][u]].x);
                        x[c] = st * 32 + u * 4 + kk < a.K ? xv : 0.f;
                    }
#pragma unroll
                    for (int r = 0; r < RTW; ++r) {
                        const float split = fmaf(fmaf((float)wl[st][r][u], SPLIT3_STEP, (float)wm[st][r][u]), SPLIT3_STEP, (float)wh[st][r][u]) * pow2f(-we[r]);
                        const float plain = __uint_as_float(__builtin_bit_cast(uintx4, u < 4 ? wh[st][r] : wm[st][r])[u & 3]);
                        const float wv = wide ? plain : split;
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], wv, acc[r][c], 0, 0, 0);
                    }
                }
        }
        // ---- results: a lane has four neighbouring columns of one output image; through LDS, so that a store takes whole
        // 256-byte runs of four images
#pragma unroll
        for (int r = 0; r < RTW; ++r) {
            const int ex = exact ? 0 : -(sx + we[r]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                floatx4_f y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[e] = ldexpf(acc[r][c][e], ex) + bj[r];
                    if (a.relu) y[e] = fmaxf(y[e], 0.f);
                }
                *reinterpret_cast<floatx4_f*>(mine + l16 * FIRST_P + 16 * c + 4 * kk) = y;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
            const auto rs = __builtin_amdgcn_make_buffer_rsrc(dst + (size_t)(r * 16) * ovox, 0, (int)FIRST_NONE, 0x00020000);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = 4 * q + kk;
                const uintx4 v = *reinterpret_cast<const uintx4*>(mine + j * FIRST_P + 4 * l16);
                const bool on = (rt0 + r) * 16 + j < a.fo;
                const unsigned o = 4u * (j * ovox + half * d.noz + zl);
                __builtin_amdgcn_raw_buffer_store_b128(v, rs, on && zl + 4 <= zn ? o : FIRST_NONE, 0, 0);
                if (d.noz & 3) {                                     // the end of a row
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        __builtin_amdgcn_raw_buffer_store_b32(v[e], rs, on && zl + 4 > zn && zl + e < zn ? o + 4 * e : FIRST_NONE, 0, 0);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        }
    }
}

// A tile length's cost in microseconds, fitted to 1500 random layers of 13 to 64 taps (tiles of each length on all of them that they
// fit; standard deviation 13 to 15 %): what a call costs; a workgroup's turns, per row tile, ... and step of 32 taps; a compute unit's
// tiles, ... and 256 staged values of them; a megabyte written.
struct FirstCost { int TZ; double call, rows, steps, tile, staged, mb; };
static const FirstCost kFirstCost[3] = {
    {128, 6.5, 0.58, 0.74, 0.28, 0.074, 0.0},
    {64, 6.3, 0.60, 0.79, 0.35, 0.070, 0.019},
    {32, 6.1, 0.52, 0.86, 0.36, 0.067, 0.042},
};

bool first_plan(int S, int f, int fo, const Dims& d, FirstPlan* P)
{
    const long long K = (long long)f * d.kx * d.ky * d.kz, vox = (long long)d.nx * d.ny * d.nz, ovox = (long long)d.nox * d.noy * d.noz;
    // (fewer taps stay with the fp32 kernel: a quarter of the layers of up to 8 are slower here)
    if (K <= 12 || K > 64 || f * vox >= (1ll << 30) - 64 || ovox >= (1ll << 26) - 64 || fo > 65535) return false;
    const int rt = (fo + 15) / 16, most = K <= 32 ? 5 : 3;
    P->nmblk = (rt + most - 1) / most; P->RTW = (rt + P->nmblk - 1) / P->nmblk;
    P->us = -1.0;
    for (const FirstCost& c : kFirstCost) {
        const int TY = 256 / c.TZ;
        const long long total = f * (long long)d.kx * (TY + d.ky - 1) * (c.TZ + d.kz - 1);
        const long long tiles = (long long)S * d.nox * ((d.noy + TY - 1) / TY) * ((d.noz + c.TZ - 1) / c.TZ);
        if (total > 256 * FIRST_NQ || tiles >= 1 << 30 || (c.TZ == 32 && d.noz >= 4096)) continue;
        const double turns = ceil((double)tiles * P->nmblk / first_slots(P->RTW)), per = (double)tiles * P->nmblk / 256;
        const double us = c.call + turns * P->RTW * (c.rows + c.steps * (K > 32 ? 2 : 1)) + per * (c.tile + c.staged * ((total + 255) / 256)) +
                          4e-6 * S * fo * ovox * c.mb;
        if (P->us >= 0 && us >= P->us) continue;
        P->us = us; P->TZ = c.TZ; P->TY = TY; P->total = (int)total; P->tiles = (int)tiles;
    }
    return P->us >= 0;
}

template <int RTW, int ST, int NQ>
static znni_status launch_first(FirstArgs a, int nmblk, hipStream_t st)
{
    const size_t lds = 4 * (2 * (size_t)((a.total + 1) & ~1) + 64 + 8 + 4 * 16 * FIRST_P);
    const int blocks = std::min(a.tiles, first_slots(RTW));
    k_direct_first<RTW, ST, NQ><<<dim3((unsigned)blocks, (unsigned)nmblk), dim3(256), lds, st>>>(a);
    return hipGetLastError() == hipSuccess ? ZNNI_OK : ZNNI_ERR_HIP;
}
template <int RTW>
static znni_status launch_rows(const FirstArgs& a, int nmblk, hipStream_t st)
{
    if (a.K <= 32)
        return a.total <= 256 * 7 ? launch_first<RTW, 1, 7>(a, nmblk, st) : launch_first<RTW, 1, FIRST_NQ>(a, nmblk, st);
    if constexpr (RTW <= 3) return launch_first<RTW, 2, FIRST_NQ>(a, nmblk, st);
    return ZNNI_ERR_SHAPE;
}

znni_status launch_direct_first(const FirstPlan& P, int f, int fo, const Dims& d, const float* in, const float* w, const float* bias,
                                float* out, int relu, hipStream_t st)
{
    FirstArgs a;
    a.in = in; a.w = w; a.bias = bias; a.out = out; a.d = d; a.f = f; a.fo = fo; a.relu = relu;
    a.taps = d.kx * d.ky * d.kz; a.K = f * a.taps;
    a.TZ = P.TZ; a.TY = P.TY; a.TYI = P.TY + d.ky - 1; a.TZI = P.TZ + d.kz - 1;
    a.tilevol = d.kx * a.TYI * a.TZI; a.total = P.total;
    a.nty = (d.noy + P.TY - 1) / P.TY; a.ntz = (d.noz + P.TZ - 1) / P.TZ; a.tiles = P.tiles;
    a.by_vol.set(a.tilevol); a.by_tz.set(a.TZI); a.by_ty.set(a.TYI); a.by_taps.set(a.taps); a.by_kz.set(d.kz); a.by_ky.set(d.ky);
    a.by_ntz.set(a.ntz); a.by_nty.set(a.nty); a.by_nox.set(d.nox);
    switch (P.RTW) {
        case 1: return launch_rows<1>(a, P.nmblk, st);
        case 2: return launch_rows<2>(a, P.nmblk, st);
        case 3: return launch_rows<3>(a, P.nmblk, st);
        case 4: return launch_rows<4>(a, P.nmblk, st);
        case 5: return launch_rows<5>(a, P.nmblk, st);
    }
    return ZNNI_ERR_SHAPE;
}

}  // namespace znni
