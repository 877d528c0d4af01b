// direct_split.hip -- direct convolution of narrow layers (few contraction slots per output) on fp16 matrix instructions.
//
// The same implicit matrix product as direct.hip, for layers whose kernel bank fits LDS.  There the fp32 matrix
// instructions and a serial stage / multiply / store sequence were the limit (8 -> 80 images of 200^3, 2^3 kernels:
// 1.84 ms, where writing the output alone takes 0.40 at the rate of a copy).  Here:
//  * products run on v_mfma_f32_16x16x32_f16 with every value split in two scaled halves, three of four partial products
//    (see mac_xd.hip; image values scaled by the largest magnitude of the staged tile, kernels by that of their output
//    image), sums fp32;
//  * workgroups are persistent: the bank is put in LDS once, and the image values of the next tile travel to registers
//    while the current one is multiplied and stored;
//  * the image values are the left operand, so that a lane holds four consecutive z of one output image and stores them
//    as 16 bytes: no transposition through LDS, no barrier between products and stores.  (One voxel per lane, sixteen
//    lanes along z: four times the store instructions, 1.07 -> 1.6 ms.)
// Before -> after: 8 -> 80 of 200^3, 2^3 1.81 -> 1.07 ms; 16 -> 16 of 128^3, 2^3 0.180 -> 0.108; 8 -> 44 of 162 x 154 x 186,
// 1 x 4 x 1 0.50 -> 0.32; 8 -> 50 of 192 x 124 x 107, 4 x 1 x 4 0.58 -> 0.30; 6 -> 12 of 100^3, 3^3 0.106 -> 0.067.  Error
// against 64 bits 0.6 to 0.8 times the former.  What bounds it: stores into rows that start anywhere (rows of 192 values
// instead of 199: 2.8 instead of 2.6 TB/s read and written) and the round trips of a tile at two waves per SIMD.
//
// Workgroup = 4 waves = one tile of TX x TY x 16*TZ16 output voxels (at most 16*CT column tiles of 16 voxels in z), all
// 16*RT output images of a row block.  Staged image tile in LDS: [hi, lo][image octet][position] units of 16 bytes, so a
// tap is a shift; a slot of the contraction is (octet, tap), four slots per matrix step.  A tile that holds values that
// are not finite is summed in plain fp32 instead (halves of an infinity are not defined).
#include <stdint.h>

#include "direct_split.h"
#include "split.h"

namespace znni {

typedef float floatx4_s __attribute__((ext_vector_type(4)));

// Column tiles per wave: what its sums and the staged values of the next tile leave room for in 256 registers.
constexpr int split_ct(int RT) { return RT <= 3 ? 4 : 2; }

struct __attribute__((packed, aligned(4))) float4_u { float x, y, z, w; };       // 16 bytes at any 4-byte address

struct SplitArgs {
    const float* in;
    const float* w;
    const half8* A;             // [row block][slot, whole steps][row tile][hi, lo][16 output images], 8 images each
    const float* rinv;          // [row blocks * 16 RT]
    const float* bias;
    float* out;
    Dims d;
    int S, f, fo, noct, nslots, nsteps;
    int TX, TY, TZ16, TYI, TZI, npos;       // tile and its staged extent
    int ntiles, relu;
    FastDiv d_tz, d_ty, d_tx, d_TZI, d_TYI, d_npos, d_TZ16, d_TY, d_taps, d_kz, d_ky;
};

// Row scales and the bank in operand layout.  grid (row tiles, parts): every workgroup of a row tile finds the scales of
// its sixteen output images again (a few thousand values from the caches).
__global__ __launch_bounds__(256) void k_split_prep(const float* __restrict__ w, half8* __restrict__ A,
                                                    float* __restrict__ rinv, int f, int fo, int taps, int noct,
                                                    int nslots4, int RT)
{
    __shared__ float mx[16][17];
    const int t = threadIdx.x, rt = blockIdx.x, jl = t >> 4, j = rt * 16 + jl;
    float m = 0.f;
    if (j < fo) {
        const float* wj = w + (size_t)j * f * taps;
        for (int e = t & 15; e < f * taps; e += 16) {
            const float v = fabsf(wj[e]);
            m = fmaxf(m, v < INFINITY ? v : 0.f);
        }
    }
    mx[jl][t & 15] = m;
    __syncthreads();
    const int jc = t & 15, js = rt * 16 + jc;           // from here on: output image along the threads
#pragma unroll
    for (int e = 0; e < 16; ++e) m = e ? fmaxf(m, mx[jc][e]) : mx[jc][0];
    const int ex = max(min(split_exp(m), 120), -120);
    if (blockIdx.y == 0 && t < 16) rinv[js] = pow2f(-ex);
    const float s = pow2f(ex);
    const int blk = rt / RT, rl = rt - blk * RT;
    for (int slot = blockIdx.y * 16 + (t >> 4); slot < nslots4; slot += gridDim.y * 16) {
        const int o = slot / taps, tap = slot - o * taps;
        half8 h, l;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = o * 8 + q;
            const float v = (o < noct && i < f && js < fo) ? w[((size_t)js * f + i) * taps + tap] : 0.f;
            _Float16 a, b;
            split2(v, s, a, b);
            h[q] = a; l[q] = b;
        }
        half8* d = A + ((size_t)blk * nslots4 + slot) * RT * 32 + rl * 32 + jc;
        d[0] = h;
        d[16] = l;
    }
}

template <int RT, int CT>
__global__ __launch_bounds__(SPLIT_NT, 2) void k_direct_split(SplitArgs a)
{
    extern __shared__ half8 lds[];
    half8* const Wl = lds;                                   // [slot][RT][hi, lo][16]
    half8* const Xs = Wl + a.nsteps * RT * 128;              // [hi, lo][noct][npos]
    int* const delta = reinterpret_cast<int*>(Xs + 2 * a.noct * a.npos);       // [4 * nsteps]
    __shared__ unsigned wmax[2][SPLIT_NT / 64];
    const Dims& d = a.d;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, l16 = lane & 15, kk = lane >> 4;
    const int mblk = blockIdx.y;
    const int taps = d.kx * d.ky * d.kz;

    {   // the bank and the slots' positions, once
        const half8* src = a.A + (size_t)mblk * a.nsteps * RT * 128;
        for (int e = t; e < a.nsteps * RT * 128; e += SPLIT_NT) Wl[e] = src[e];
        for (int e = t; e < 4 * a.nsteps; e += SPLIT_NT) {
            // (slots past the last one hold zero kernels and read the last tap's place)
            const unsigned sl = (unsigned)min(e, a.nslots - 1), o = a.d_taps.div(sl), tap = sl - o * a.d_taps.d;
            const unsigned ab = a.d_kz.div(tap), c = tap - ab * a.d_kz.d, aa = a.d_ky.div(ab), b = ab - aa * a.d_ky.d;
            delta[e] = (int)o * a.npos + ((d.kx - 1 - (int)aa) * a.TYI + (d.ky - 1 - (int)b)) * a.TZI + (d.kz - 1 - (int)c);
        }
    }
    // unit u of this thread: (octet, position); worked out again where it is used (registers are what is short)
    auto unit_octet = [&](int u, unsigned& p) {
        const unsigned e = min((unsigned)(t + SPLIT_NT * u), (unsigned)(a.noct * a.npos - 1)), o = a.d_npos.div(e);
        p = e - o * a.d_npos.d;
        return (int)o;
    };
    // column tiles of this wave
    int vx[CT], vy[CT], vz[CT], vox[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const unsigned ct = (unsigned)(wave * CT + c), xy = a.d_TZ16.div(ct), x = a.d_TY.div(xy);
        vz[c] = (int)(ct - xy * a.d_TZ16.d) * 16; vx[c] = (int)x; vy[c] = (int)(xy - x * a.d_TY.d);
        if (vx[c] >= a.TX) { vx[c] = -1; vy[c] = vz[c] = 0; }                 // beyond the tile: nothing to store
        vox[c] = (max(vx[c], 0) * a.TYI + vy[c]) * a.TZI + vz[c] + l16;
    }
    float rj[RT], bj[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int j = (mblk * RT + r) * 16 + l16;
        rj[r] = a.rinv[j];
        bj[r] = a.bias ? a.bias[min(j, a.fo - 1)] : 0.f;
    }

    // Tiles: every XCD (consecutive workgroups go to the eight of them in turn) walks a contiguous range, z fastest, its
    // workgroups side by side, so that halos and partly written cache lines meet in one L2.
    const int xcd = blockIdx.x & 7, nw = (int)(gridDim.x >> 3), w0 = (int)(blockIdx.x >> 3);
    const int per = (a.ntiles + 7) >> 3, tend = min((xcd + 1) * per, a.ntiles);
    int tile = xcd * per + w0;
    const size_t nvox = (size_t)d.nx * d.ny * d.nz;
    const size_t ovox = (size_t)d.nox * d.noy * d.noz;
    auto origin = [&](int tl, int& s, int& x0, int& y0, int& z0) {
        const unsigned q = a.d_tz.div((unsigned)tl), q2 = a.d_ty.div(q);
        z0 = (tl - (int)(q * a.d_tz.d)) * a.TZ16 * 16; y0 = (int)(q - q2 * a.d_ty.d) * a.TY;
        s = (int)a.d_tx.div(q2); x0 = ((int)q2 - s * (int)a.d_tx.d) * a.TX;
    };
    float raw[SPLIT_UNITS][8];
    auto load = [&](int tl) {
        int s, x0, y0, z0;
        origin(tl, s, x0, y0, z0);
        const float* img = a.in + (size_t)s * a.f * nvox;
#pragma unroll
        for (int u = 0; u < SPLIT_UNITS; ++u) {
            if (SPLIT_NT * u >= a.noct * a.npos) break;
            unsigned p;
            const int o = unit_octet(u, p);
            const unsigned xy = a.d_TZI.div(p), lx = a.d_TYI.div(xy);
            const int gx = min(x0 + (int)lx, d.nx - 1), gy = min(y0 + (int)(xy - lx * a.d_TYI.d), d.ny - 1);
            const int gz = min(z0 + (int)(p - xy * a.d_TZI.d), d.nz - 1);
            const float* v = img + (size_t)((gx * d.ny + gy) * d.nz + gz);
#pragma unroll
            for (int q = 0; q < 8; ++q) raw[u][q] = v[(size_t)min(8 * o + q, a.f - 1) * nvox];
        }
    };
    // largest magnitude of this thread's values
    float m;
    auto magnitude = [&]() {
        m = 0.f;
#pragma unroll
        for (int u = 0; u < SPLIT_UNITS; ++u)
            if (SPLIT_NT * u < a.noct * a.npos)
#pragma unroll
                for (int q = 0; q < 8; q += 2) max3_abs(m, raw[u][q], raw[u][q + 1]);
    };
    if (tile < tend) load(tile);
    for (int it = 0; tile < tend; tile += nw, ++it) {
        magnitude();
        auto largest = [&](unsigned (&w)[SPLIT_NT / 64]) {
            const unsigned v = wave_max(m);
            if (lane == 0) w[wave] = v;
            __syncthreads();
            unsigned b = w[0];
#pragma unroll
            for (int e = 1; e < SPLIT_NT / 64; ++e) b = max(b, w[e]);
            return b;
        };
        unsigned mb = largest(wmax[it & 1]);                 // (also: the previous tile has been multiplied)
        const bool plain = mb >= 0x7f800000u;
        const float sx = plain ? 0.f : pow2f(split_exp(__uint_as_float(mb)));
        const float inv = plain ? 0.f : pow2f(-split_exp(__uint_as_float(mb)));
        if (!plain)
#pragma unroll
            for (int u = 0; u < SPLIT_UNITS; ++u) {
                if (t + SPLIT_NT * u >= a.noct * a.npos) break;
                unsigned p;
                const int o = unit_octet(u, p);
                half8 h, l;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    _Float16 x, y;
                    split2(raw[u][q], 8 * o + q < a.f ? sx : 0.f, x, y);
                    h[q] = x; l[q] = y;
                }
                Xs[t + SPLIT_NT * u] = h;
                Xs[a.noct * a.npos + t + SPLIT_NT * u] = l;
            }
        __syncthreads();
        if (tile + nw < tend) load(tile + nw);

        int s, x0, y0, z0;
        origin(tile, s, x0, y0, z0);
        floatx4_s acc[RT][CT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[r][c] = floatx4_s{0.f, 0.f, 0.f, 0.f};
        if (!plain) {
            for (int st = 0; st < a.nsteps; ++st) {
                const half8* xs = Xs + delta[4 * st + kk];
                half8 xh[CT], xl[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) { xh[c] = xs[vox[c]]; xl[c] = xs[a.noct * a.npos + vox[c]]; }
                const half8* wl = Wl + (4 * st + kk) * RT * 32 + l16;
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const half8 wh = wl[r * 32], wo = wl[r * 32 + 16];
#pragma unroll
                    for (int c = 0; c < CT; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xl[c], wh, acc[r][c], 0, 0, 0);
#pragma unroll
                    for (int c = 0; c < CT; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh[c], wo, acc[r][c], 0, 0, 0);
#pragma unroll
                    for (int c = 0; c < CT; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh[c], wh, acc[r][c], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int j = (mblk * RT + r) * 16 + l16;
            if (j >= a.fo) continue;
            float* oj = a.out + ((size_t)s * a.fo + j) * ovox;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int X = x0 + vx[c], Y = y0 + vy[c], Z = z0 + vz[c] + 4 * kk;
                if (vx[c] < 0 || X >= d.nox || Y >= d.noy || Z >= d.noz) continue;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[r][c][e] * inv * rj[r];
                if (plain) {
                    for (int e = 0; e < min(4, d.noz - Z); ++e) {
                        float sum = 0.f;
                        for (int i = 0; i < a.f; ++i)
                            for (int q = 0; q < taps; ++q) {
                                const int cz = q % d.kz, b = (q / d.kz) % d.ky, aa = q / (d.kz * d.ky);
                                sum = fmaf(a.w[((size_t)j * a.f + i) * taps + q],
                                           a.in[((size_t)s * a.f + i) * nvox +
                                                (size_t)(((X + d.kx - 1 - aa) * d.ny + Y + d.ky - 1 - b) * d.nz + Z + e + d.kz - 1 - cz)],
                                           sum);
                            }
                        if (e == 0) v[0] = sum; else if (e == 1) v[1] = sum; else if (e == 2) v[2] = sum; else v[3] = sum;
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] += bj[r];
                    if (a.relu) v[e] = fmaxf(v[e], 0.f);
                }
                float* o = oj + ((size_t)X * d.noy + Y) * d.noz + Z;
                if (Z + 3 < d.noz) {
                    *reinterpret_cast<float4_u*>(o) = float4_u{v[0], v[1], v[2], v[3]};
                } else {
                    o[0] = v[0];
                    if (Z + 1 < d.noz) o[1] = v[1];
                    if (Z + 2 < d.noz) o[2] = v[2];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------ host side
// Tile of at most `cols` column tiles: the one that wastes least, counting column slots (matrix work and stores) and
// staged units; ties go to the longer rows.
static bool split_tile(const Dims& d, int noct, int cols, int max_units, SplitPlan* P)
{
    double best = -1.0;
    const int zu = (d.noz + 15) / 16;
    for (int tx = 1; tx <= 4; ++tx)
        for (int ty = 1; ty <= 8; ++ty) {
            const int tzmax = cols / (tx * ty);
            if (tzmax < 1) continue;
            const int nz = (zu + tzmax - 1) / tzmax, tz = (zu + nz - 1) / nz;
            if (tz < (zu < 2 ? zu : 2)) continue;           // (runs of at least 128 bytes)
            const long long npos = (long long)(tx + d.kx - 1) * (ty + d.ky - 1) * (16 * tz + d.kz - 1);
            if (npos * noct > max_units) continue;
            const double tiles = (double)((d.nox + tx - 1) / tx) * ((d.noy + ty - 1) / ty) * nz;
            const double cost = tiles * (cols * 16.0 + 0.5 * noct * npos);
            if (best < 0 || cost < best * 0.999) {
                best = cost;
                P->TX = tx; P->TY = ty; P->TZ16 = tz; P->npos = (int)npos; P->nz = nz;
            }
        }
    return best > 0;
}

bool split_plan(int S, int f, int fo, const Dims& d, SplitPlan* P)
{
    const long long taps = (long long)d.kx * d.ky * d.kz;
    P->noct = (f + 7) / 8;
    const long long nslots = taps * P->noct;
    if (nslots > 256) return false;
    const int rt = (fo + 15) / 16, nblk = (rt + 4) / 5;
    P->RT = (rt + nblk - 1) / nblk;
    P->nmblk = nblk;
    P->CT = split_ct(P->RT);
    P->nslots = (int)nslots;
    P->nsteps = (int)((nslots + 3) / 4);
    if (P->nmblk > 65535 || (size_t)P->nsteps * P->RT * 2048 > 40 * 1024) return false;
    // fewer than five images leave most of an octet empty; fp32 products are level there
    if (f < 5) return false;
    if (!split_tile(d, P->noct, SPLIT_NT / 64 * P->CT, SPLIT_NT * SPLIT_UNITS, P)) return false;
    const long long tiles = (long long)S * ((d.nox + P->TX - 1) / P->TX) * ((d.noy + P->TY - 1) / P->TY) * P->nz;
    if (tiles > (1 << 30)) return false;
    P->ntiles = (int)tiles;
    P->lds = (size_t)P->nsteps * P->RT * 2048 + (size_t)2 * P->noct * P->npos * 16 + (size_t)16 * P->nsteps;
    P->bytes = (size_t)P->nmblk * P->nsteps * P->RT * 2048 + (size_t)P->nmblk * P->RT * 64;
    return true;
}

template <int RT>
static znni_status launch_rt(const SplitArgs& a, const SplitPlan& P, hipStream_t st)
{
    const void* fn = (const void*)k_direct_split<RT, split_ct(RT)>;
    if (P.lds > 48 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P.lds) != hipSuccess)
        return ZNNI_ERR_HIP;
    // two workgroups per CU; a multiple of eight, so that every XCD has the same number
    const int per = (P.ntiles + 7) / 8, nw = per < 64 ? per : 64;
    k_direct_split<RT, split_ct(RT)><<<dim3(8 * nw, P.nmblk), dim3(SPLIT_NT), P.lds, st>>>(a);
    return hipGetLastError() != hipSuccess ? ZNNI_ERR_HIP : ZNNI_OK;
}

znni_status launch_direct_split(const SplitPlan& P, int S, int f, int fo, const Dims& d, const float* in, const float* w,
                                const float* bias, float* out, int relu, void* workspace, hipStream_t st)
{
    half8* A = (half8*)workspace;
    float* rinv = (float*)((char*)workspace + (size_t)P.nmblk * P.nsteps * P.RT * 2048);
    const int taps = d.kx * d.ky * d.kz, nslots4 = 4 * P.nsteps;
    const int parts = (nslots4 + 15) / 16;
    k_split_prep<<<dim3(P.nmblk * P.RT, parts), dim3(256), 0, st>>>(w, A, rinv, f, fo, taps, P.noct, nslots4, P.RT);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    SplitArgs a;
    a.in = in; a.w = w; a.A = A; a.rinv = rinv; a.bias = bias; a.out = out;
    a.d = d; a.S = S; a.f = f; a.fo = fo; a.noct = P.noct; a.nslots = P.nslots; a.nsteps = P.nsteps;
    a.TX = P.TX; a.TY = P.TY; a.TZ16 = P.TZ16;
    a.TYI = P.TY + d.ky - 1; a.TZI = 16 * P.TZ16 + d.kz - 1; a.npos = P.npos;
    a.ntiles = P.ntiles; a.relu = relu;
    a.d_tz.set(P.nz); a.d_ty.set((d.noy + P.TY - 1) / P.TY); a.d_tx.set((d.nox + P.TX - 1) / P.TX);
    a.d_TZI.set(a.TZI); a.d_TYI.set(a.TYI); a.d_npos.set(P.npos); a.d_TZ16.set(P.TZ16); a.d_TY.set(P.TY);
    a.d_taps.set(taps); a.d_kz.set(d.kz); a.d_ky.set(d.ky);
    switch (P.RT) {
        case 1: return launch_rt<1>(a, P, st);
        case 2: return launch_rt<2>(a, P, st);
        case 3: return launch_rt<3>(a, P, st);
        case 4: return launch_rt<4>(a, P, st);
        case 5: return launch_rt<5>(a, P, st);
    }
    return ZNNI_ERR_SHAPE;
}

}  // namespace znni
