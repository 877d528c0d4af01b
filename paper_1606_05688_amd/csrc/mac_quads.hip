// mac_quads.hip -- multiply-accumulate without x transform for rows that lie in blocks of four x, tile pairs (passes_tiles.hip).
//
// The contraction, the split of values in two scaled halves, the chunks of sixteen images and what is done about values far apart
// are those of mac_xd.hip.  What differs is who works on what.  Rows along x lie in blocks of four, a block of every oy after the
// other, so four neighbouring pencils share every line of 128 bytes, and a wave that reads its own pencil's rows uses a
// quarter of each: 48 -> 48 of 320^3, 5^3 kernels had 265 million lines on their way to the vector L1 caches for 80 million lines of
// spectra, and the kernel took 4.9 of its 6.3 ms without a single product.  So here the four waves of a workgroup are four
// neighbouring pencils of one strip: they read whole lines together (a wave per image quad; of a load's lanes sixteen hold a line,
// four x of four pencils) and leave every pencil's values in its part of LDS under that pencil's own scale, which is found by
// LDS atomics behind one barrier a chunk.  Every wave has kernel operands of its own then, and reads them straight into the
// registers of a matrix step, two steps ahead; they come from L2, where the strips and inputs of a pencil meet them.  (Through LDS,
// shared by four strips of one pencil as in mac_xd.hip, they were the reason for a wave to be a strip.)  No barrier but the
// two of a chunk is left.  Results leave through buffer stores that drop what is out of range: without a branch, a 64-bit product
// and two multiplications for each, 650 vector instructions of a wave became 150.
//
// Against mac_xd.hip's kernel on the same rows: 40 -> 40 of 128^3, 3^3 at length 36 352 -> 315 us; 48 -> 48 of 160^3, 5^3 at 56 929 -> 856;
// of 320^3 at 84 6300 -> 5870; 37 -> 45 of 93 x 110 x 131, 3 x 4 x 5 at 32 290 -> 255.
//
// What bounds it, at the lengths that are picked (counters; share of the time that a SIMD's matrix pipe is busy, that it issues other
// vector instructions, that the bytes would take at copy speed; waves a SIMD):
//   48 -> 48 of 320^3, 5^3, length 36 (6855 us)                41 %   32 %   38 %   1.8   1.93 GHz
//   40 -> 40 of 128^3, 3^3, length 28 (317)                    25     26     45     1.9   2.32
//   37 -> 45 of 93 x 110 x 131, 3 x 4 x 5, length 32 (269)     22     25     41     1.9   2.26
//   48 -> 48 of 160^3, 5^3, length 56, first turn (541)        35     35            2.9   2.08
// The three add up to the time: with two or three waves a SIMD they hardly overlap, and where a strip has more than six tiles the
// next chunk's rows are only requested when the chunk begins.  (With them on their way to LDS while one is multiplied,
// global_load_lds, the 320^3 layer at length 84 took 6120 instead of 5870 us: the kernel operands behind them return in order.
// Neighbouring quads on one XCD changed nothing.)
#include <algorithm>
#include "mac_xd.h"

namespace znni {

// LDS of a workgroup: per pencil [hi, lo][image quad][x] units of sixteen bytes, two pencils four banks of sixteen bytes apart so
// that the lanes of a store, four x of each, meet no bank twice.
constexpr int q_xw(int CT) { return 16 * CT + 16; }          // pitch of an image quad's row of staged units
constexpr int q_ps(int CT) { return 8 * q_xw(CT) + 4; }      // ... of a pencil's
template <int RT, int CT>
constexpr size_t q_lds_bytes() { return (size_t)16 * (4 * q_ps(CT) + 4 * RT) + 4 * 32; }
// Workgroups per CU: what 256, 168 or 128 registers a lane allow.
template <int RT, int CT>
constexpr int q_blocks()
{
    if (RT * CT <= 2) return 4;
    return RT * CT <= 6 ? 3 : 2;
}

// split_conj with a scale for either part
__device__ __forceinline__ void split_pair(float x, float y, float sx, float sy, unsigned& hi, unsigned& lo)
{
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(hi) : "v"(x), "v"(sx));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(hi) : "v"(y), "v"(sy));
    asm("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(lo) : "v"(x), "v"(sx), "v"(hi));
    asm("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(lo) : "v"(y), "v"(sy), "v"(hi));
}

// (A function of its own: written as the kernel, three by four tiles spill; 48 -> 48 of 320^3, 5^3 12.2 -> 12.35 ms.)
template <int RT, int CT>
__device__ __forceinline__ void q_body(const XdArgs& g, half8* lds)
{
    constexpr int XW = q_xw(CT), PS = q_ps(CT), NR = CT + 1;
    // (three by two tiles with one set: three workgroups a CU, 912 -> 856 us for 48 -> 48 of 160^3, 5^3)
    constexpr bool DB = RT <= 3 && !(RT == 3 && CT == 2);    // two sets of kernel operands, or one that is refilled row group by row group
    constexpr int RG = DB ? RT : RT == 5 ? 3 : 2;
    constexpr bool AHEAD = RT * CT <= 6;
    half8* const Xs = lds;                                   // [pencil][hi, lo][quad][XW]
    float* const rjs = reinterpret_cast<float*>(lds + 4 * PS);
    unsigned* const red = reinterpret_cast<unsigned*>(rjs + 16 * RT);        // [turn][largest, smallest][pencil], [pencil]

    const unsigned xcd = blockIdx.x & 7, bslot = blockIdx.x >> 3;
    const unsigned qg = g.d_sub.div(bslot), sub = bslot - qg * g.d_sub.d;
    const int pq = (int)(qg * 8 + xcd);
    if (pq >= g.npencils) return;
    const int mblk = (int)g.d_nwg.div(sub), strip = (int)sub - mblk * (int)g.d_nwg.d;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int l16 = lane & 15, kk = lane >> 4;
    const int sI = (int)g.d_spr.div((unsigned)strip);
    const int col0 = (strip - sI * (int)g.d_spr.d) * 16 * CT;
    const int K = g.K, f = g.f;
    const int poz = (int)g.d_Ny.div((unsigned)pq), oy0 = (pq - poz * (int)g.d_Ny.d) * 4;
    const bool live = oy0 + wave < g.Ny;
    const int poy = min(oy0 + wave, g.Ny - 1);
    const bool mirror = poz >= g.zc;
    const int aoz = mirror ? g.Nz - poz : poz, aoy = mirror && poy ? g.Ny - poy : poy;

    if (t < 32) red[t] = (t & 4) && t < 24 ? ~0u : 0u;
    // ---- kernel operands, straight into the registers of a step
    const int nslots = K * ((f + 3) >> 2), nsteps = (nslots + 3) >> 2;
    const int sstride = 2 * g.Mp;
    const half8* const Ab = g.A + (size_t)(aoz * g.Ny + aoy) * nslots * sstride + mblk * RT * 32;
    half8 ah[DB ? 2 : 1][RT], al[DB ? 2 : 1][RT];
    auto load_a = [&](half8 (&h)[RT], half8 (&l)[RT], int step, int r0, int r1) {
        const unsigned off = (unsigned)(min(4 * step + kk, nslots - 1) * sstride + l16) * 16u;

        const half8* p = reinterpret_cast<const half8*>(reinterpret_cast<const char*>(Ab) + off);
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (r >= r0 && r < r1) { h[r] = p[r * 32]; l[r] = p[r * 32 + 16]; }
    };

    floatx4 re[RT][CT], im[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) { re[r][c] = floatx4{0.f, 0.f, 0.f, 0.f}; im[r][c] = re[r][c]; }

    // ---- image rows: of a round's lanes sixteen hold a block of four x of four pencils, one line of memory
    const int so = (lane >> 2) & 3;
    const float2* const xin = g.X2 + (size_t)(unsigned)(sI * f) * g.ximg + (size_t)poz * g.xpen;
    const int xlast = min(g.nx, col0 + 16 * CT + K - 1) - 1;
    const int xpen0 = 4 * min(oy0 + so, g.Ny - 1);
    auto xoff = [&](int x) { x = min(x, xlast); return (x >> 2) * g.xblk + (x & 3); };
    const int RB = K > 1 ? CT + 1 : CT;
    int chunk = 0, QC = 4, sexp = 126, lexp = 126;          // exponents of the scales: of this wave's pencil, of a lane's staged one
    bool apart = false;
    unsigned most = 0;
    float2 raw[NR][4];
    // image quad and round of this wave's n-th unit of a chunk of qc quads (surplus units repeat the last one)
    auto unit = [&](int n, int qc, int& q, int& r) {
        if (qc == 4) { q = wave; r = min(n, RB - 1); return; }
        const int u = min(wave + 4 * n, qc * RB - 1);
        if (qc == 3) { r = u / 3; q = u - 3 * r; }
        else { r = qc == 2 ? u >> 1 : u; q = qc == 2 ? u & 1 : 0; }
    };
    auto request = [&]() {
        const int i0 = chunk * 16, qc = min(4, ((f + 3) >> 2) - 4 * chunk);
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            int q, r;
            unit(n, qc, q, r);
            const unsigned off = 8u * (unsigned)(xoff(col0 + 16 * r + 4 * kk + (lane & 3)) + xpen0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                raw[n][e] = *reinterpret_cast<const float2*>(
                    reinterpret_cast<const char*>(xin + (size_t)(unsigned)min(i0 + 4 * q + e, f - 1) * g.ximg) + off);
        }
    };
    auto quad_max = [&](unsigned v) {
        v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));
        return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));
    };
    auto stage = [&]() {
        float m = 0.f;
        unsigned mn = ~0u;
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            float u = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) max3_abs(u, raw[n][e].x, raw[n][e].y);
            m = fmaxf(m, u);
            mn = min(mn, small_code(u));
        }
        const int turn = chunk % 3;
        unsigned* const rd = red + 8 * turn;
        const unsigned qm = quad_max(__float_as_uint(m)), qn = ~quad_max(~mn);
        if ((lane & 3) == 0) { atomicMax(rd + so, qm); atomicMin(rd + 4 + so, qn); }
        __syncthreads();                                     // (also: all waves are through with the chunk before)
        unsigned mine = rd[wave], sm = rd[4 + wave], their = rd[so];
        const unsigned any = max(max(rd[0], rd[1]), max(rd[2], rd[3]));
        if (__builtin_amdgcn_readfirstlane((int)any) >= 0x7f800000) {        // infinities or NaNs: the scale is that of the finite values
            if (t < 4) red[24 + t] = 0;
            m = 0.f;
#pragma unroll
            for (int n = 0; n < NR; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (hidden from the compiler, which would otherwise look at every value of every chunk before it branches)
                    asm volatile("" : "+v"(raw[n][e].x), "+v"(raw[n][e].y));
                    const float ax = fabsf(raw[n][e].x), ay = fabsf(raw[n][e].y);
                    max3_abs(m, ax < INFINITY ? ax : 0.f, ay < INFINITY ? ay : 0.f);
                }
            __syncthreads();
            const unsigned qf = quad_max(__float_as_uint(m));
            if ((lane & 3) == 0) atomicMax(red + 24 + so, qf);
            __syncthreads();
            mine = red[24 + wave]; their = red[24 + so];
        }
        if (t < 8) red[8 * ((turn + 2) % 3) + t] = t & 4 ? ~0u : 0u;         // (last read before this chunk's first barrier)
        mine = (unsigned)__builtin_amdgcn_readfirstlane((int)mine);
        sm = (unsigned)__builtin_amdgcn_readfirstlane((int)sm);
        // next to the largest value of all chunks so far, whose scale it carries
        most = max(most, mine);
        apart |= split_too_wide(most, sm);
        const int sn = min(sexp, split_exp(__uint_as_float(mine)));
        if (sn < sexp && chunk) {                            // a larger chunk: the sums follow its scale
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        re[r][c][e] = ldexpf(re[r][c][e], sn - sexp);
                        im[r][c][e] = ldexpf(im[r][c][e], sn - sexp);
                    }
        }
        sexp = sn;
        lexp = min(lexp, split_exp(__uint_as_float(their)));
        const float sx = pow2f(lexp), sy = mirror ? sx : -sx;
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            int q, r;
            unit(n, QC, q, r);
            uintx4 h, l;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                unsigned a, b;
                split_pair(raw[n][e].x, raw[n][e].y, sx, sy, a, b);
                h[e] = a; l[e] = b;
            }
            half8* d = Xs + so * PS + q * XW + 16 * r + 4 * kk + (lane & 3);
            d[0] = __builtin_bit_cast(half8, h);
            d[4 * XW] = __builtin_bit_cast(half8, l);
        }
        __syncthreads();
        ++chunk;
    };

    // position in the contraction: steps left in the chunk, and this lane group's slot (quad of the chunk, tap)
    int left = 0, quad = 0, a = 0, qx = 0;
    const half2 turn_x = mirror ? half2{(_Float16)1.f, (_Float16)-1.f} : half2{(_Float16)-1.f, (_Float16)1.f};
    auto swp = [](half8 v, half2 s) {
        half8 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const half2 p = half2{v[2 * e + 1], v[2 * e]} * s;
            o[2 * e] = p[0]; o[2 * e + 1] = p[1];
        }
        return o;
    };
    const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
#define ZNNI_Q_MFMA(D, A, X, C) D = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, X, C, 0, 0, 0)
    auto step = [&](half8 (&h)[RT], half8 (&l)[RT], int gs) {
        if (left == 0) {                                     // next chunk of up to sixteen images
            QC = min(4, ((f + 3) >> 2) - 4 * chunk);
            left = (K * QC + 3) >> 2;
            quad = QC == 4 ? kk : QC == 3 ? (kk == 3 ? 0 : kk) : kk & (QC - 1);
            a = QC == 4 ? 0 : QC == 3 ? (kk == 3) : kk >> (QC - 1);
            qx = quad * XW;
            if (chunk && !AHEAD) request();
            stage();
            if (AHEAD && 16 * chunk < f) request();
        }
        --left;
        const half8* const xs = Xs + wave * PS + l16 + qx + max(K - 1 - a, 0);
        if (QC == 4) ++a;
        else {
            quad += QC == 3; a += QC == 3 ? 1 : QC == 2 ? 2 : 4;
            if (quad >= QC) { quad -= QC; ++a; }
            qx = quad * XW;
        }
        if (4 * gs + 3 >= nslots) {                          // slots past the last one count as zeros
            const bool on = 4 * gs + kk < nslots;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                uintx4 u = __builtin_bit_cast(uintx4, h[r]), v = __builtin_bit_cast(uintx4, l[r]);
#pragma unroll
                for (int e = 0; e < 4; ++e) { u[e] = on ? u[e] : 0u; v[e] = on ? v[e] : 0u; }
                h[r] = __builtin_bit_cast(half8, u); l[r] = __builtin_bit_cast(half8, v);
            }
        }
        if constexpr (2 * RT > CT) {
#pragma unroll
            for (int r0 = 0; r0 < RT; r0 += RG) {
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const half8 hr = xs[16 * c], lr = xs[4 * XW + 16 * c];
                    const half8 hi = swp(hr, turn_x), li = swp(lr, turn_x);
                    floatx4 tr[RG], ti[RG];
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_Q_MFMA(tr[r - r0], h[r], lr, zero); ZNNI_Q_MFMA(ti[r - r0], h[r], li, zero); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_Q_MFMA(tr[r - r0], l[r], hr, tr[r - r0]); ZNNI_Q_MFMA(ti[r - r0], l[r], hi, ti[r - r0]); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_Q_MFMA(tr[r - r0], h[r], hr, tr[r - r0]); ZNNI_Q_MFMA(ti[r - r0], h[r], hi, ti[r - r0]); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { re[r][c] += tr[r - r0]; im[r][c] += ti[r - r0]; }
                }
                if constexpr (!DB) load_a(h, l, gs + 1, r0, r0 + RG);
            }
        } else {
            half8 bh[RT], bl[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) { bh[r] = swp(h[r], -turn_x); bl[r] = swp(l[r], -turn_x); }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const half8 hr = xs[16 * c], lr = xs[4 * XW + 16 * c];
                floatx4 tr[RT], ti[RT];
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_Q_MFMA(tr[r], h[r], lr, zero); ZNNI_Q_MFMA(ti[r], bh[r], lr, zero); }
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_Q_MFMA(tr[r], l[r], hr, tr[r]); ZNNI_Q_MFMA(ti[r], bl[r], hr, ti[r]); }
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_Q_MFMA(tr[r], h[r], hr, tr[r]); ZNNI_Q_MFMA(ti[r], bh[r], hr, ti[r]); }
#pragma unroll
                for (int r = 0; r < RT; ++r) { re[r][c] += tr[r]; im[r][c] += ti[r]; }
            }
        }
    };
#undef ZNNI_Q_MFMA
    request();
    load_a(ah[0], al[0], 0, 0, RT);
    if constexpr (DB) load_a(ah[1], al[1], 1, 0, RT);
    if (t < RT * 16) rjs[t] = g.rinv[mblk * RT * 16 + t];
    __syncthreads();
    if constexpr (DB) {
        // (the last step of an odd number by itself: a second step that might not run would have the first one's operands waited
        // for as if they were the youngest)
        int gs = 0;
        for (; gs + 1 < nsteps; gs += 2) {
            step(ah[0], al[0], gs);
            load_a(ah[0], al[0], gs + 2, 0, RT);
            step(ah[1], al[1], gs + 1);
            load_a(ah[1], al[1], gs + 3, 0, RT);
        }
        if (gs < nsteps) step(ah[0], al[0], gs);
    } else {
        for (int gs = 0; gs < nsteps; ++gs) step(ah[0], al[0], gs);
    }
    if (!live) return;

    // Kernels of an output image of uneven size: every image counts by itself, next to the largest value of all (read again for it).
    const float2* const xrow = xin + 4 * poy;
    const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    unsigned bits = __float_as_uint(rjs[min(ln, RT * 16 - 1)]);
    if (RT > 4) bits |= __float_as_uint(rjs[64 + l16]);
    const bool uneven = __ballot((int)bits < 0) != 0;
    if (uneven && !apart) {
        // (where some kernels are far below the largest and not zero, halves hold those badly, and an image that is zero is as
        // good as one that is far below the others)
        const unsigned tiny = __ballot(bits & 1u) != 0;
        unsigned mn = ~0u;
        for (int i = 0; i < f; ++i) {
            const float2* row = xrow + (size_t)(unsigned)i * g.ximg;
            for (int x = ln; x < 16 * CT + K - 1; x += 64) {
                const float2 v = row[xoff(col0 + x)];
                float m = 0.f;
                max3_abs(m, v.x, v.y);
                mn = min(mn, (__float_as_uint(m) << 1) - 1u + tiny);
            }
        }
        apart = split_too_wide(most, wave_min(mn));
    }

    if (apart) {
        // All over again in fp32, from global memory, four slots of one complex image each per pair of matrix instructions
        // (kernels: their two halves added up, or, where an output image's are uneven, the sum along y again).
        const float sx = pow2f(sexp);
        const size_t per = (size_t)K * g.fp * g.Mp;
        const float2* const a1 = g.A1 + (size_t)aoz * g.ky * per + mblk * RT * 16 + l16;
        auto again = [&](int r, int i, int tap) {
            float2 s = make_float2(0.f, 0.f);
            for (int b = 0, t = 0; b < g.ky; ++b) {          // t = (aoy * b) mod Ny
                s = cfma(s, a1[b * per + ((size_t)tap * g.fp + i) * g.Mp + r * 16], g.tw[t]);
                t += aoy;
                if (t >= g.Ny) t -= g.Ny;
            }
            const float cr = g.row[(mblk * RT + r) * 16 + l16] * g.scale, ci = g.cinv[i];
            return make_float2(s.x * cr * ci, s.y * cr * ci);
        };
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) { re[r][c] = zero; im[r][c] = zero; }
        for (int gs = 0; gs < nsteps; ++gs) {
            const int sl = min(4 * gs + kk, nslots - 1);
            int qd, tap;
            xd_slot(sl, K, (f + 3) >> 2, qd, tap);
            const half8* ap = Ab + (size_t)sl * sstride + l16;
            const float on = 4 * gs + kk < nslots ? sx : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float cs = 4 * qd + q < f ? on : 0.f;
                const float2* row = xrow + (size_t)(unsigned)min(4 * qd + q, f - 1) * g.ximg;
                float2 x[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const float2 v = row[xoff(col0 + c * 16 + l16 + K - 1 - tap)];
                    x[c] = make_float2(v.x * cs, v.y * cs);
                }
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const half2 hh = reinterpret_cast<const half2*>(ap + r * 32)[q], hl = reinterpret_cast<const half2*>(ap + r * 32 + 16)[q];
                    float ar = (float)hh[0] + (float)hl[0], ai = (float)hh[1] + (float)hl[1];
                    if (uneven) { const float2 e = again(r, 4 * qd + q, tap); ar = e.x; ai = e.y; }
                    ai = mirror ? -ai : ai;
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        re[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, x[c].x, re[r][c], 0, 0, 0);
                        im[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, x[c].y, im[r][c], 0, 0, 0);
                        re[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai, -x[c].y, re[r][c], 0, 0, 0);
                        im[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai, x[c].x, im[r][c], 0, 0, 0);
                    }
                }
            }
        }
    }

    // ---- results: element e of lane (kk, l16) is image 4 kk + e, output l16.  Rows of Yd are padded to whole fours.  (Buffer
    // stores: lanes out of range write nothing, without a branch for every one of them.)
    constexpr unsigned NONE = 0x80000000u;
    const size_t yimg = (size_t)g.yimg * 8;
    float2* const ypen = g.Yd + (size_t)(unsigned)(sI * g.fo) * g.yimg + (size_t)poz * g.ypen + (size_t)poy * 4;
    unsigned off[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int xo = col0 + c * 16 + l16;
        off[c] = xo < g.nox ? (unsigned)((xo >> 2) * g.yblk + (xo & 3)) * 8u + (unsigned)(4 * kk) * (unsigned)yimg : NONE;
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int j0 = (mblk * RT + r) * 16;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (j0 + e >= g.fo) break;
            const int ex = (int)(__float_as_uint(rjs[r * 16 + 4 * kk + e]) >> 23 & 255u) - 127 - sexp;
            const auto row = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(ypen) + (size_t)(unsigned)(j0 + e) * yimg, 0, (int)NONE, 0x00020000);
            const unsigned none = j0 + e + 4 * kk < g.fo ? 0u : NONE;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int o = (int)(off[c] | none);
                const float2 v = make_float2(ldexpf(re[r][c][e], ex), ldexpf(im[r][c][e], ex));
                typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), row, o, 0, 0);
            }
        }
    }
}

template <int RT, int CT>
__global__ __launch_bounds__(256, (q_blocks<RT, CT>())) void k_mac_tiles(XdArgs g)
{
    extern __shared__ half8 lds[];
    q_body<RT, CT>(g, lds);
}

template <int RT, int CT>
static znni_status launch_q(const LayerPlan& L, XdArgs g, hipStream_t st)
{
    const Dims& d = L.d;
    const int spr = ((d.nox + 15) / 16 + CT - 1) / CT, quads = (d.Ny + 3) / 4;
    g.nstrips = L.S * spr; g.npencils = d.Nz * quads;        // (quads of pencils)
    g.d_sub.set((unsigned)(g.nstrips * L.mac_nmblk)); g.d_spr.set((unsigned)spr); g.d_nwg.set((unsigned)g.nstrips);
    g.d_Ny.set((unsigned)quads);
    const long long blocks = (long long)((g.npencils + 7) / 8) * 8 * g.nstrips * L.mac_nmblk;
    if (blocks > 0x7fffffffll) return ZNNI_ERR_SHAPE;
    constexpr size_t lds = q_lds_bytes<RT, CT>();
    void (*kernel)(XdArgs) = k_mac_tiles<RT, CT>;
    if (lds > 48 * 1024 && hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return ZNNI_ERR_HIP;
    kernel<<<dim3((unsigned)blocks), dim3(256), lds, st>>>(g);
    return hipGetLastError() == hipSuccess ? ZNNI_OK : ZNNI_ERR_HIP;
}

// Widest strip of a row block: accumulators, operands and a chunk on its way in 256 registers.
static constexpr int q_max_ct(int RT) { return RT <= 2 ? 5 : 7 - RT; }

// The strip width whose waves are through a chunk first: products, rounds of staging, what a wave waits for in any case (in
// cycles of a SIMD).  It does not look at the number of inputs, so that turns take the whole layer's width.
int quads_strip(const LayerPlan& L)
{
    const int tiles = (L.d.nox + 15) / 16, RT = L.mac_RTW;
    int CT = 1;
    long long best = -1;
    for (int c = 1; c <= q_max_ct(RT); ++c) {
        const long long n = (long long)((tiles + c - 1) / c) * (96 * L.d.kx * RT * c + 200 * (c + 1) + 800);
        if (best < 0 || n <= best) { best = n; CT = c; }
    }
    return CT;
}

template <int RT>
static znni_status launch_q_cols(const LayerPlan& L, const XdArgs& g, hipStream_t st)
{
    constexpr int MAXCT = q_max_ct(RT);
    switch (quads_strip(L)) {
        case 1: return launch_q<RT, 1>(L, g, st);
        case 2: return launch_q<RT, 2>(L, g, st);
        case 3: if constexpr (MAXCT >= 3) return launch_q<RT, 3>(L, g, st); break;
        case 4: if constexpr (MAXCT >= 4) return launch_q<RT, 4>(L, g, st); break;
        case 5: if constexpr (MAXCT >= 5) return launch_q<RT, 5>(L, g, st); break;
    }
    return ZNNI_ERR_SHAPE;
}

znni_status launch_mac_quads(const LayerPlan& L, const XdArgs& g, hipStream_t st)
{
    switch (L.mac_RTW) {
        case 1: return launch_q_cols<1>(L, g, st);
        case 2: return launch_q_cols<2>(L, g, st);
        case 3: return launch_q_cols<3>(L, g, st);
        case 4: return launch_q_cols<4>(L, g, st);
        case 5: return launch_q_cols<5>(L, g, st);
    }
    return ZNNI_ERR_SHAPE;
}

}  // namespace znni
