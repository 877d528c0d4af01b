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
// Before -> after: 8 -> 80 of 200^3, 2^3 1.80 -> 0.96 ms; 16 -> 16 of 128^3, 2^3 0.175 -> 0.101; 8 -> 44 of 162 x 154 x 186,
// 1 x 4 x 1 0.50 -> 0.31; 6 -> 12 of 100^3, 3^3 0.104 -> 0.072; with one voxel of 1e9 in every 100 000: 1.00, 0.116, 0.32, 0.078.  Error
// against 64 bits 0.6 to 0.8 times the former.  What bounds it: stores into rows that start anywhere (rows of 192 values
// instead of 199: 2.8 instead of 2.6 TB/s read and written) and the round trips of a tile at two waves per SIMD.
//
// Workgroup = 4 waves = one tile of TX x TY x 16*TZ16 output voxels (at most 16*CT column tiles of 16 voxels in z), all
// 16*RT output images of a row block.  Staged image tile in LDS: [hi, lo][image octet][position] units of 16 bytes, so a
// tap is a shift; a slot of the contraction is (octet, tap), four slots per matrix step.
//
// Halves cover 2^40: a value far below the largest of its tile would lose bits to a neighbour that its outputs never meet
// (one voxel of 1e9 among ones: 1e-3 of all results of its tile).  So a tile whose magnitudes lie too far apart, or that
// holds infinities, is staged in fp32, in the same place (eight images are 32 bytes either way), and multiplied on the fp32
// instructions; so are all tiles where the kernel values of an output image lie too far apart (k_split_prep).
#include <stdint.h>

#include "direct_split.h"
#include "split.h"

namespace znni {

typedef float floatx4_s __attribute__((ext_vector_type(4)));

// Column tiles per wave: what its sums and the staged values of the next tile leave room for in 256 registers.
constexpr int split_ct(int RT) { return RT <= 3 ? 4 : 2; }

typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));           // 16 bytes at any 4-byte address

struct SplitArgs {
    const float* in;
    const float* w;
    const half8* A;             // [row block][slot, whole steps][row tile][hi, lo][16 output images], 8 images each
    // [row blocks * 16 RT] inverse scales of the kernels (powers of two: the upper half of a float), negative where the row
    // tile is in fp32
    const unsigned short* rinv;
    int* next;                  // [row blocks][8] tiles handed out per XCD beyond the first three of every workgroup
    const float* bias;
    float* out;
    Dims d;
    int S, f, fo, noct, nslots, nsteps;
    int TX, TY, TZ16, TYI, TZI, npos;       // tile and its staged extent
    int ntiles, relu;
    FastDiv d_tz, d_ty, d_tx, d_TZI, d_TYI, d_npos, d_TZ16, d_TY, d_taps, d_kz, d_ky;
};

// Row scales and the bank in operand layout.  grid (row tiles, parts): every workgroup of a row tile finds the scales of
// its sixteen output images again, from their kernel values in LDS (40 KB at most).  A row tile whose kernel values halves
// do not hold has its bank in fp32, two times 16 bytes for eight images either way: one with an infinity, or where all taps
// of an input image, or one tap of all of them, lie below the range of the largest.  (A single small value is no reason:
// next to others of its image and its tap it adds less to an output than their rounding.)
__global__ __launch_bounds__(256) void k_split_prep(const float* __restrict__ w, half8* __restrict__ A,
                                                    unsigned short* __restrict__ rinv, int* __restrict__ next, int f,
                                                    int fo, int taps, int nslots4,
                                                    int RT)
{
    extern __shared__ float wl[];                       // [16][f][taps]
    __shared__ int ex16[16], wide;
    const int t = threadIdx.x, rt = blockIdx.x, jl = t >> 4, jc = t & 15, row = f * taps;
    const size_t all = (size_t)fo * row, w0 = (size_t)rt * 16 * row;
    for (int e = t; e < 16 * row; e += 256) wl[e] = w0 + e < all ? w[w0 + e] : 0.f;
    if (t == 0) wide = 0;
    if (blockIdx.y == 0 && t < 8 && rt % RT == 0) next[rt / RT * 8 + t] = 0;
    __syncthreads();
    const float* wj = wl + jl * row;
    float m = 0.f;
    unsigned mn = ~0u;
    int plain = 0;
    // largest finite magnitude of n values
    auto group = [&](const float* p, int n, int step) {
        float g = 0.f;
        for (int q = 0; q < n; ++q) {
            const float v = fabsf(p[q * step]);
            plain |= v == INFINITY;
            g = fmaxf(g, v < INFINITY ? v : 0.f);
        }
        return g;
    };
    for (int i = jc; i < f; i += 16) {
        const float g = group(wj + i * taps, taps, 1);
        m = fmaxf(m, g);
        mn = min(mn, small_code(taps > 1 ? g : 8.f * g));        // (a single tap is a single value, small by chance now and then)
    }
    for (int q = jc; q < taps; q += 16) mn = min(mn, small_code(group(wj + q, f, taps)));
#pragma unroll
    for (int o = 8; o; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o));
        mn = min(mn, (unsigned)__shfl_xor((int)mn, o));
    }
    if (plain || split_too_wide(__float_as_uint(m), mn)) wide = 1;
    if (jc == 0) ex16[jl] = split_exp(m);
    __syncthreads();
    if (blockIdx.y == 0 && t < 16) rinv[rt * 16 + t] = (unsigned short)((127 - ex16[t]) << 7 | wide << 15);
    const float s = pow2f(ex16[jc]);                    // from here on: output image along the threads
    const int blk = rt / RT, rl = rt - blk * RT;
    for (int slot = blockIdx.y * 16 + (t >> 4); slot < nslots4; slot += gridDim.y * 16) {
        const int o = slot / taps, tap = slot - o * taps;
        half8 h, l;
        floatx4_s v4[2];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = o * 8 + q;
            const float v = i < f ? wl[jc * row + i * taps + tap] : 0.f;
            _Float16 a, b;
            split2(v, s, a, b);
            h[q] = a; l[q] = b;
            v4[q >> 2][q & 3] = v * s;
        }
        if (wide) {
            h = __builtin_bit_cast(half8, v4[0]);
            l = __builtin_bit_cast(half8, v4[1]);
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
    __shared__ unsigned wred[2][2][SPLIT_NT / 64];           // [turn][largest, smallest][wave]
    const Dims& d = a.d;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, l16 = lane & 15, kk = lane >> 4;
    const int mblk = blockIdx.y;

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
    unsigned rj[RT];
    float bj[RT];
    unsigned wide = 0;                                       // bit r: kernels of row tile r in fp32
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int j = (mblk * RT + r) * 16 + l16;
        rj[r] = a.rinv[j];
        wide |= (reinterpret_cast<const unsigned*>(a.rinv)[(mblk * RT + r) * 8] >> 15 & 1u) << r;     // (one address: a scalar load)
        bj[r] = a.bias ? a.bias[min(j, a.fo - 1)] : 0.f;
    }

    // Tiles: every XCD (consecutive workgroups go to the eight of them in turn) walks a contiguous range, z fastest, its
    // workgroups side by side, so that halos and partly written cache lines meet in one L2.  From three row tiles on a
    // workgroup takes its fourth and later tiles from a counter: with a fixed stride one that was held up (a tile in fp32)
    // stays behind the others for good, and the lines no longer meet (8 -> 80 of 200^3, 2^3, normally distributed values:
    // 1.17 ms, 0.96 from the counter).  With one or two row tiles a tile is short, and the counter costs more than it
    // saves (16 -> 16 of 128^3, 2^3: 0.101 ms, 0.118 from the counter).
    constexpr bool DYN = RT >= 3;
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
    // largest magnitude of this thread's values, and the smallest one's code
    float m;
    unsigned mn;
    auto magnitude = [&]() {
        m = 0.f;
        mn = ~0u;
#pragma unroll
        for (int u = 0; u < SPLIT_UNITS; ++u)
            if (SPLIT_NT * u < a.noct * a.npos)
#pragma unroll
                for (int q = 0; q < 8; q += 2) {
                    max3_abs(m, raw[u][q], raw[u][q + 1]);
                    mn = min(min(mn, small_code(raw[u][q])), small_code(raw[u][q + 1]));
                }
    };
    int tile1 = tile + nw, taken = tile1 + nw;               // the next tile, and (thread 0) the one after it
    __shared__ int snext[2];
    if (tile < tend) load(tile);
    for (int it = 0; tile < tend; ++it) {
        magnitude();
        unsigned (&red)[2][SPLIT_NT / 64] = wred[it & 1];
        {
            const unsigned vx = wave_max(m), vn = wave_min(mn);
            if (lane == 0) { red[0][wave] = vx; red[1][wave] = vn; }
            if (DYN && t == 0) snext[it & 1] = taken;
        }
        __syncthreads();                                     // (also: the previous tile has been multiplied)
        unsigned mb = red[0][0], sm = red[1][0];
#pragma unroll
        for (int e = 1; e < SPLIT_NT / 64; ++e) { mb = max(mb, red[0][e]); sm = min(sm, red[1][e]); }
        mb = (unsigned)__builtin_amdgcn_readfirstlane((int)mb);
        sm = (unsigned)__builtin_amdgcn_readfirstlane((int)sm);
        const bool plain = wide != 0 || mb >= 0x7f800000u || split_too_wide(mb, sm);
        // (in fp32 the largest goes to 2^94: no sum overflows whose result does not, and 2^-127 of it is a normal number)
        const int sexp = plain ? min(split_exp(__uint_as_float(mb)) + 80, 126) : split_exp(__uint_as_float(mb));
        const float sx = pow2f(sexp), inv = pow2f(-sexp);
#pragma unroll
        for (int u = 0; u < SPLIT_UNITS; ++u) {
            if (t + SPLIT_NT * u >= a.noct * a.npos) break;
            unsigned p;
            const int o = unit_octet(u, p);
            half8 h, l;
            if (!plain) {
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    _Float16 x, y;
                    split2(raw[u][q], 8 * o + q < a.f ? sx : 0.f, x, y);
                    h[q] = x; l[q] = y;
                }
            } else {
                floatx4_s v[2];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q >> 2][q & 3] = 8 * o + q < a.f ? raw[u][q] * sx : 0.f;
                h = __builtin_bit_cast(half8, v[0]);
                l = __builtin_bit_cast(half8, v[1]);
            }
            Xs[t + SPLIT_NT * u] = h;
            Xs[a.noct * a.npos + t + SPLIT_NT * u] = l;
        }
        __syncthreads();
        if (tile1 < tend) load(tile1);
        const int tile2 = DYN ? __builtin_amdgcn_readfirstlane(snext[it & 1]) : tile1 + nw;
        if (DYN && t == 0) taken = xcd * per + 3 * nw + atomicAdd(a.next + mblk * 8 + xcd, 1);

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
        } else {
            for (int sl = 0; sl < a.nslots; ++sl) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {                // four images a matrix instruction, one per lane group
                    const float* xs = reinterpret_cast<const float*>(Xs + h * a.noct * a.npos + delta[sl]) + kk;
                    float x[CT];
#pragma unroll
                    for (int c = 0; c < CT; ++c) x[c] = xs[4 * vox[c]];
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const half8* wl = Wl + (sl * RT + r) * 32 + l16;
                        const _Float16* hw = reinterpret_cast<const _Float16*>(wl) + 4 * h + kk;
                        const float wv = wide >> r & 1 ? reinterpret_cast<const float*>(wl + 16 * h)[kk] : (float)hw[0] + (float)hw[128];
#pragma unroll
                        for (int c = 0; c < CT; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], wv, acc[r][c], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int j = (mblk * RT + r) * 16 + l16;
            if (j >= a.fo) continue;
            float* oj = a.out + ((size_t)s * a.fo + j) * ovox;
            // the smaller factor first: either alone may be out of range where the result is not
            const float rv = __uint_as_float((rj[r] & 0x7fffu) << 16), f0 = fminf(inv, rv), f1 = fmaxf(inv, rv);
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int X = x0 + vx[c], Y = y0 + vy[c], Z = z0 + vz[c] + 4 * kk;
                // vmcnt(4): a wave's stores in flight, held back so that partly written lines meet (8 -> 44 of 162 x 154 x
                // 186, 1 x 4 x 1: 0.313 ms, 0.324 without)
                if constexpr (CT == 4) __builtin_amdgcn_s_waitcnt(0x0f74);
                if (vx[c] < 0 || X >= d.nox || Y >= d.noy || Z >= d.noz) continue;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = acc[r][c][e] * f0 * f1 + bj[r];
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
        tile = tile1;
        tile1 = tile2;
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

// What a call costs; for every 512 tiles (two a compute unit, and a tile at least) the products, the staged values and the steps'
// latency; the kernels' preparation; megabytes written and read.  Fitted to 1634 random layers (standard deviation 16 %).
double split_us(const SplitPlan& P, int S, int f, int fo, const Dims& d)
{
    const double turns = (P.ntiles > 512 ? P.ntiles / 512.0 : 1.0) * P.nmblk, pairs = P.RT * P.CT;
    const double out = 4e-6 * S * fo * ((double)d.nox * d.noy * d.noz), in = 4e-6 * S * f * ((double)d.nx * d.ny * d.nz) * P.nmblk;
    return 10.7 + turns * (pairs * (0.155 + 0.0358 * P.nsteps) + 0.40 * P.noct * P.npos / 256 + 0.30 * P.nsteps) + 0.097 * P.nsteps * P.noct +
           0.19 * out + 0.064 * in;
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
    unsigned short* rinv = (unsigned short*)((char*)workspace + (size_t)P.nmblk * P.nsteps * P.RT * 2048);
    int* next = (int*)(rinv + P.nmblk * P.RT * 16);
    const int taps = d.kx * d.ky * d.kz, nslots4 = 4 * P.nsteps;
    const int parts = (nslots4 + 15) / 16;
    k_split_prep<<<dim3(P.nmblk * P.RT, parts), dim3(256), (size_t)64 * f * taps, st>>>(w, A, rinv, next, f, fo, taps, nslots4, P.RT);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    SplitArgs a;
    a.in = in; a.w = w; a.A = A; a.rinv = rinv; a.next = next; a.bias = bias; a.out = out;
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
