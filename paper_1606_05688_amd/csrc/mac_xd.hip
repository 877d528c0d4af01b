// mac_xd.hip -- multiply-accumulate for layers whose x axis is never transformed.
//
// For one input of the batch the work of the last kernel-transform stage plus the per-bin multiply-accumulate
// (Algorithm 3, second stage; kernel transform pruned as in Section III-A) is, per (oz, oy) pencil,
//
//     Yt[j][ox] = sum_{(i,a)} A(a,i,j) * exp(-2 pi i a ox / Nx) * Xt[i][ox],
//
// a contraction of length f*kx per bin.  The inverse x transform of that product, kept on the valid outputs
// xo = 0 .. nx-kx (Section III-B), is exactly the kx-tap valid convolution along x
//
//     Yd[j][xo] = sum_{(i,a)} A(a,i,j) * X2[i][xo + kx-1 - a],
//
// where X2 is the image transformed along z and y only: the same contraction length per output, with no x
// transform on either side and no twiddle products.  So when every kernel-spectrum value would be used once
// (few inputs per batch) the x axis is never transformed: the forward x pass, the inverse x pass and the tensors
// between them disappear, and the right operand of the matrix product is the image row itself, read at kx
// shifted offsets.  (With many inputs per batch a kernel-spectrum value generated once per bin serves them all, as in
// mac_batch.hip, but on fp32 products and behind two more passes: batches of small images come here as well.)
//
// Layers whose planes are cut into tiles (passes_tiles.hip) go through mac_quads.hip instead, with the same halves, scales and
// kernel operands; here are the others: whole planes, four at a time or by separate passes.
//
// Layouts: X2[img][oz][oy][x < ldx] as the forward y pass leaves it, Yd[imgo][oz][oy][xo < ldxo], which the inverse y pass
// reads with a transposing load; or, next to the fused z+y kernels that take four planes (passes_fused.hip), X2[img][oz]
// [x/4][oy][x%4] and Yd likewise (k_mac_planes).  A: see k_kprep_xd.
//
// The products run on the fp16 matrix instructions (v_mfma_f32_16x16x32_f16, sixteen times the rate of the fp32 ones)
// with every fp32 value carried as two halves, v = hi + lo (two halves together hold 22 bits and a sign, an error of
// about 1.5 fp32 roundings), and three of the four partial products kept: hi hi, hi lo, lo hi (the fourth is below
// 2^-22 of the first).  Sums stay fp32.  Halves have a narrow exponent range, so both operands are scaled by powers
// of two, which costs no accuracy: the image values of a wave's strip by their largest magnitude so far (the sums are
// rescaled when a later chunk is larger), the kernel transforms of an output image by a bound of theirs.  With the
// largest value at 2^14, every value down to 2^-17 of it keeps all 22 bits, smaller ones an absolute error of 2^-40 of
// the largest.
//
// Values that lie further apart than that:
//  * Input images whose kernels make up for another magnitude (a network that is not normalised): half of the distance
//    between the kernels of the images moves to their values, so that both sides stay in range (kprep_row_scale in mac.hip;
//    images up to 2^40 apart come out to 32-bit accuracy).  The forward y pass does that to the values on its way out:
//    done here as they are staged, it cost the small layers 1 us more (12 -> 5 of 49 x 38 x 41, 3 x 2 x 5 kernels 40.2
//    against 39.5 us for the layer, 3 x 5 -> 13 of 56 x 50 x 68, 5 x 5 x 1 86.3 against 84.1; 8 -> 8 of 64^3, 5^3 55.9
//    against 57.0).
//  * Values along x: the x axis is not transformed, so a row next to one large value has outputs that never meet it.  A
//    wave whose largest values at some x lie more than 2^SPLIT_SPAN below the largest of its strip so far sums all over again
//    in fp32, from global memory.  (A voxel of 1e9 in every 100 000: 40 -> 40 of 128^3, 3^3 kernels 0.84 -> 1.34 ms for the layer, 80 -> 80
//    with 7^3 2.9 -> 6.8; on fp32 products alone 0.95 and 4.2.)
//  * Kernels of an output image of uneven size (the sums of their magnitudes more than 2^14 apart, or zero: kprep_row_scale
//    leaves two bits behind).  Elsewhere the largest input images have a part in every output image, and what is lost of the
//    others is small next to it.  Here an output image may be made of the small ones alone: every image then counts by
//    itself when a wave looks at how far its values lie apart, and the fp32 sums take kernel transforms made again from A1.
//    (8 x 40 -> 20 of 40 x 24 x 22, groups of images 2^30 apart that no output image shares: 2.9e-3 off without it, 3e-7
//    with it.  Where kernels are even it costs at most 1 % of the layer.)
//  * What is left: single taps along x far below the others of their output image (an absolute error of 2^-40 of the largest).
//
// Whole layers come out 0.6 to 1.0 times as far from their 64-bit values as with fp32 matrix
// instructions (80 -> 80 of 128^3, 7^3 kernels: 3.7e-7 against 5.4e-7), and the kernel is (multiply-accumulate alone,
// before and after): 80 -> 80 of 128^3, 7^3 2.53 -> 1.05 ms; 40 -> 40 of 128^3, 3^3 0.37 -> 0.22; 37 -> 45 of 93 x 110 x
// 131, 3 x 4 x 5 0.33 -> 0.25; 80 -> 80 of 200^3, 5^3 9.1 -> 3.8.  Up to eight images with one or two taps it is level to a
// fifth behind (7 -> 38 of 126 x 180 x 119, 1 tap: 0.118 -> 0.142): there nothing but reading and writing spectra is left.
// What bounds it: at 48 -> 48 of 320^3, 5^3 on whole planes (5.0 ms, 6.3 with workgroup-wide staging and 64-column tiles of four waves) the
// matrix pipes are busy half of the time at 1.75 GHz, where the passes next to it run at 2.1 to 2.2: power, of which the
// products take most.  Without image reads it took 4.3 ms, without stores 4.4, without any memory access 3.7, with a third
// of the products 3.7; requesting the next chunk's cache lines ahead, other wave priorities and fewer vector
// instructions while staging changed nothing.  At 40 -> 40 of 128^3, 3^3 (0.22 ms, 4.8 TB/s) and at 80 -> 80 of 128^3, 7^3
// (1.05 ms, 4.3 GB of which 3 are kernel transforms) it is memory.
//
// Complex products as real ones: with the contraction running over (image, real / imaginary part), the kernel
// operand (Ar, Ai) meets (Xr, -Xi) for the real part of the result and (Xi, Xr) for the imaginary part.  The first is what
// is staged, the second is made of it with one packed instruction per register.
//
// A wave owns a strip of 16*CT outputs along x of one pencil (oz, oy) of one input and RT row tiles of 16 output images; the
// four waves of a workgroup own four strips of a pencil, of one input or of several, and share its kernel operands (and, with
// one row tile or narrow strips of one input, the staged rows: xd_shared).  Strips
// are as wide as the row divides best into (launch_xd_cols_s): rows of 316 outputs are four strips of 80 where four waves
// of one 192-wide tile and the next left a sixth of the products to padding.  Input images go through in chunks of sixteen.  A wave
// reads its own rows into registers, splits them and leaves them in its own part of LDS as [image quad][x] units of 16
// bytes, the operand layout, so that a tap is a shift by one unit; no wave waits for another's rows (a workgroup that
// staged together met at two barriers a chunk).  One matrix step contracts four (quad, tap) slots: sixteen images of one tap,
// or, in a last chunk of fewer images, several taps of fewer quads.  Kernel operands travel global memory -> registers -> LDS,
// requested two pairs of steps and parked one pair ahead, one quarter per wave (every wave reading all of them for itself
// asks more of the vector L1 than it delivers: 85 / CT bytes per clock of 64); one barrier per pair of steps.
#include <algorithm>
#include "mac_xd.h"

namespace znni {


// One row tile, and narrow strips: the four waves take neighbouring strips of one input and stage them together.  With one row
// tile there is little to multiply and the image rows are what counts; in narrow strips the columns that two of them share are as
// many as their own.  Together a wave reads whole rows of four images, and shared columns are read once (19 -> 5 of 295^3, 5^3
// kernels 935 us, every wave its own strip 1210; 14 -> 12 of 111 x 88 x 87, 6 x 2 x 4 43 against 45; 28 -> 75 of 62^3, 7^3 107
// against 117).  Three to five row tiles of two column tiles are slower that way (277 layers: level, 1.2 and 1.2 % of the layer).
constexpr bool xd_shared(int RT, int CT, bool planes) { return (RT == 1 || CT == 1 || (RT == 2 && CT == 2)) && !planes; }
template <int RT, int CT, bool PLANES>
constexpr size_t xd_lds_bytes()
{
    return (size_t)16 * ((xd_shared(RT, CT, PLANES) ? 8 * (64 * CT + 16) : 4 * 8 * (16 * CT + 16)) + 4 * 128 * RT + 4 * RT + 5);
}
// Workgroups per CU: five of the smallest tiles (held to 96 registers a lane), three where LDS and registers (168) allow, two
// otherwise.
template <int RT, int CT, bool PLANES>
constexpr int xd_blocks()
{
    if (xd_shared(RT, CT, PLANES) && RT == 1 && CT <= 2) return 5;
    return xd_lds_bytes<RT, CT, PLANES>() <= 53 * 1024 && RT * CT <= 6 ? 3 : 2;
}

// What lanes of a wave have written to LDS is there for its other lanes: the wave's LDS operations complete in order, so that
// nothing has to be waited for, and the fences keep the compiler from moving any across.
__device__ __forceinline__ void wave_handover()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int RT, int CT, bool SUM, bool PLANES>
__device__ __forceinline__ void xd_body(const XdArgs& g, half8* lds)
{
    // staged columns of a strip (its outputs and their halo) and the pitch of an image quad (rows start on the same bank:
    // the sixteen-lane groups of a 16-byte LDS read then share no bank in any phase)
    constexpr bool SHARED = xd_shared(RT, CT, PLANES);
    constexpr int XN = 16 * CT + 8, XW = (SHARED ? 64 : 16) * CT + 16;
    // Rounds of a wave over a strip's units: strips of three column tiles and more take a quad per round (its image rows are
    // then scalar addresses) and the columns beyond 64 of all quads in further ones.
    // Staged together, wave w takes quad w, 64 columns a round and the halo in a last one.
    constexpr int XH = CT >= 3 ? (XN > 64 ? XN - 64 : 0) : XN, NQ = CT >= 3 ? 4 : 0, NR = SHARED ? CT + 1 : NQ + (4 * XH + 63) / 64;
    // Whether the four sums of an accumulator are neighbouring outputs of one image, stored as 32 bytes a lane, or outputs
    // of four images, stored as 128 bytes of an image by sixteen lanes.  The latter takes 2 to 3 % less from three row tiles
    // on and in planes (8 x 32 -> 32 of 64^3, 7^3 0.26 against 0.30 ms), the former below (7 -> 9 of 150 x 142 x 95 57 against 60 us).
    constexpr bool XROWS = RT <= 2 && !PLANES;
    // Where registers allow, the first chunk's rows are requested before anything is waited for, and the rows of the next
    // chunk while one is multiplied.
    constexpr bool MORE = RT > 1 || CT >= 3;                // (elsewhere another wave per SIMD is worth more)
    constexpr bool EARLY = MORE && RT * CT <= 10, AHEAD = MORE && RT <= 2 && RT * CT <= 8;
    static_assert(XD_MAX_K - 1 <= 8, "the halo is eight columns");
    half8* const As = lds;                                   // [two pairs of steps][slot kk][row tile][hi, lo][16]

    // (the integer divisions of a workgroup's start cost as much as a matrix step: high products instead)
    const unsigned xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const unsigned qg = g.d_sub.div(slot), rem = slot - qg * g.d_sub.d;
    const unsigned sub = g.d_pg.div(rem);
    const int pencil = (int)((qg * 8 + xcd) * g.d_pg.d + (rem - sub * g.d_pg.d));
    if (pencil >= g.npencils) return;
    const int mblk = (int)g.d_nwg.div(sub);
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int l16 = lane & 15, kk = lane >> 4;
    const int strip = SHARED ? (int)sub - mblk * (int)g.d_nwg.d : ((int)sub - mblk * (int)g.d_nwg.d) * 4 + wave;
    const bool live = strip < g.nstrips;                     // (waves without a strip only carry kernel operands)
    const int sI = (int)g.d_spr.div((unsigned)min(strip, g.nstrips - 1));
    const int row0 = (min(strip, g.nstrips - 1) - sI * (int)g.d_spr.d) * (SHARED ? 64 : 16) * CT;       // first staged column
    const int wcol = SHARED ? wave * 16 * CT : 0, col0 = row0 + wcol;                                   // ... and this wave's first
    const int K = g.K, f = g.f;
    const int poz = (int)g.d_Ny.div((unsigned)pencil), poy = pencil - poz * g.Ny;
    half8* const Xs = lds + 4 * RT * 128 + (SHARED ? 0 : wave * 8 * XW);      // this wave's own, or all waves': [hi, lo][quad][XW]
    float* const rjs = reinterpret_cast<float*>(lds + 4 * RT * 128 + (SHARED ? 8 : 32) * XW);           // [RT * 16]
    unsigned* const wred = reinterpret_cast<unsigned*>(rjs + RT * 16);        // [turn][largest, smallest][wave], [wave]

    // ---- kernel operands: this thread's share of a step, NU units of 16 bytes (surplus units repeat the last one).
    // Slots past the last one are read from it.
    const int nslots = K * ((f + 3) >> 2), nsteps = (nslots + 3) >> 2;
    const int sstride = 2 * g.Mp, slast = (nslots - 1) * sstride;       // (32 bits: the layer call's shape limits)
    constexpr int NU = (RT + 1) / 2;
    const half8* Ab = g.A + (size_t)pencil * nslots * sstride + mblk * RT * 32;
    int u_off[NU], u_rest[NU], u_e[NU];                      // offset of the unit's slot in the step requested next
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        u_e[i] = min(wave + 4 * i, 2 * RT - 1) * 64 + lane;
        const int sl = u_e[i] / (RT * 32);
        u_off[i] = sl * sstride;
        u_rest[i] = u_e[i] - sl * (RT * 32);
    }
    half8 ring[2][NU];                                       // a pair of steps
    auto load_a = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                ring[h][i] = *reinterpret_cast<const half8*>(reinterpret_cast<const char*>(Ab) +
                                                             (size_t)(unsigned)(min(u_off[i], slast) + u_rest[i]) * 16);
                u_off[i] = min(u_off[i], slast) + 4 * sstride;
            }
    };
    // The pair's operands to LDS; slots past the last one become zeros (only the last pair can hold any).
    auto park_a = [&](int step, int buf) {
        half8* d = As + buf * RT * 256;
        if (4 * step + 7 >= nslots) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < NU; ++i) {
                    half8 v = ring[h][i];
                    if (4 * (step + h) + u_e[i] / (RT * 32) >= nslots)
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = (_Float16)0;
                    d[h * RT * 128 + u_e[i]] = v;
                }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < NU; ++i) d[h * RT * 128 + u_e[i]] = ring[h][i];
        }
    };

    floatx4 re[RT][CT], im[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) { re[r][c] = floatx4{0.f, 0.f, 0.f, 0.f}; im[r][c] = re[r][c]; }

    load_a();

    const float2* xrow = g.X2 + (size_t)(unsigned)(sI * f) * g.ximg + (size_t)poz * g.xpen + (size_t)poy * g.xrow;
    const int xlast = min(g.nx, row0 + (SHARED ? 64 : 16) * CT + K - 1) - 1;     // last column any of the strip's outputs needs
    auto xoff = [&](int x) { x = min(x, xlast); return (x >> 2) * g.xblk + (x & 3); };
    int QC = 4;                                              // image quads of the chunk
    // image quad and column of this lane's unit in round n (surplus lanes repeat the last one)
    auto rest = [&](int n) { return min(lane + 64 * (n - NQ), 4 * XH - 1); };
    auto unit_q = [&](int n) {
        if (SHARED) return wave;
        return n < NQ ? n : rest(n) / max(XH, 1);
    };
    auto unit_x = [&](int n) {
        if (SHARED) return n < CT ? 64 * n + lane : 64 * CT + (lane & 7);
        return n < NQ ? min(lane, XN - 1) : (NQ ? 64 : 0) + rest(n) % max(XH, 1);
    };
    int sexp = 126;                                          // exponent of the scale the image values carry
    int chunk = 0;
    bool apart = false;                                      // magnitudes along x too far apart for halves
    unsigned most = 0;                                       // largest finite magnitude (its bits) of the chunks so far
    // One chunk of sixteen images of the strip to LDS, a (quad, x) unit per lane and round.  Values beyond a row are read
    // from its end, images beyond the last from the last: neither reaches a stored output (the images count as zeros).
    // whether round n holds any of the chunk's qc image quads
    auto round = [&](int n, int qc) {
        if (SHARED) return wave < qc;
        return n < NQ ? n < qc : 64 * (n - NQ) < qc * XH;
    };
    float2 raw[NR][4];
    auto request = [&]() {
        const int i0 = chunk * 16, qc = min(4, ((f + 3) >> 2) - 4 * chunk);
        // (rounds of quads beyond the last image are neither read nor staged: no lane group's slot names them)
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            if (!round(n, qc)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) raw[n][q] = make_float2(0.f, 0.f);
                continue;
            }
            const int uq = unit_q(n);
            const unsigned off = 8u * (unsigned)xoff(row0 + unit_x(n));
#pragma unroll
            for (int q = 0; q < 4; ++q)
                raw[n][q] = *reinterpret_cast<const float2*>(
                    reinterpret_cast<const char*>(xrow + (size_t)(unsigned)min(i0 + 4 * uq + q, f - 1) * g.ximg) + off);
        }
    };
    auto stage = [&]() {
        const int i0 = chunk * 16;
        // largest magnitude, and the code of the smallest: of the images of a unit together, since their products
        // are added up (an image far below the others, say of rounding errors only, is no reason to leave halves)
        float m = 0.f;
        unsigned mn = ~0u;
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            float u = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) max3_abs(u, raw[n][q].x, raw[n][q].y);
            m = fmaxf(m, u);
            mn = min(mn, small_code(u));
        }
        unsigned mb = wave_max(m), sm = wave_min(mn);
        if constexpr (SHARED) {
            unsigned* const red = wred + (chunk & 1) * 8;
            if (lane == 0) { red[wave] = mb; red[4 + wave] = sm; }
            __syncthreads();                                 // (also: all waves are through with the chunk before)
            mb = (unsigned)__builtin_amdgcn_readfirstlane((int)max(max(red[0], red[1]), max(red[2], red[3])));
            sm = (unsigned)__builtin_amdgcn_readfirstlane((int)min(min(red[4], red[5]), min(red[6], red[7])));
        }
        if (mb >= 0x7f800000u) {                             // infinities or NaNs: the scale is that of the finite values
            m = 0.f;
#pragma unroll
            for (int n = 0; n < NR; ++n)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // (hidden from the compiler, which would otherwise look at every value of every chunk before it branches)
                    asm volatile("" : "+v"(raw[n][q].x), "+v"(raw[n][q].y));
                    const float ax = fabsf(raw[n][q].x), ay = fabsf(raw[n][q].y);
                    max3_abs(m, ax < INFINITY ? ax : 0.f, ay < INFINITY ? ay : 0.f);
                }
            mb = wave_max(m);
            if constexpr (SHARED) {
                if (lane == 0) wred[16 + wave] = mb;
                __syncthreads();
                mb = (unsigned)__builtin_amdgcn_readfirstlane((int)max(max(wred[16], wred[17]), max(wred[18], wred[19])));
                __syncthreads();
            }
        }
        // next to the largest value of all chunks so far, whose scale it carries
        most = max(most, mb);
        apart |= split_too_wide(most, sm);
        const int sn = min(sexp, split_exp(__uint_as_float(mb)));
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
        const float sx = pow2f(sn);
        if constexpr (!SHARED) wave_handover();              // (all lanes are through with the chunk before)
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            if (!round(n, QC)) continue;
            const int uq = unit_q(n);
            uintx4 h, l;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned a, b;
                split_conj(raw[n][q].x, raw[n][q].y, i0 + 4 * uq + q < f ? sx : 0.f, a, b);
                h[q] = a; l[q] = b;
            }
            half8* d = Xs + uq * XW + unit_x(n);
            d[0] = __builtin_bit_cast(half8, h);
            d[4 * XW] = __builtin_bit_cast(half8, l);
        }
        if constexpr (SHARED) __syncthreads();
        else wave_handover();
        ++chunk;
    };

    // position in the contraction: steps left in the chunk, and this lane group's slot (quad of the chunk, tap)
    int left = 0, quad = 0, a = 0, qx = 0;                   // qx = quad * XW
    auto step = [&](const half8* as) {                       // as: this lane group's kernel operands of the step
        if (left == 0) {                                     // next chunk of up to sixteen images
            QC = min(4, ((f + 3) >> 2) - 4 * chunk);
            left = (K * QC + 3) >> 2;
            quad = QC == 4 ? kk : QC == 3 ? (kk == 3 ? 0 : kk) : kk & (QC - 1);
            a = QC == 4 ? 0 : QC == 3 ? (kk == 3) : kk >> (QC - 1);
            qx = quad * XW;
            if (!(chunk ? AHEAD : EARLY)) request();
            stage();
            if (AHEAD && 16 * chunk < f) request();
        }
        --left;
        const half8* xs = Xs + wcol + l16 + qx + max(K - 1 - a, 0);
        if (QC == 4) ++a;
        else {
            quad += QC == 3; a += QC == 3 ? 1 : QC == 2 ? 2 : 4;
            if (quad >= QC) { quad -= QC; ++a; }
            qx = quad * XW;
        }
        half8 ah[RT], al[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) { ah[r] = as[r * 32]; al[r] = as[r * 32 + 16]; }
        // (r, -i) -> (i, r), or of the kernel operand (r, i) -> (i, -r): one packed instruction per register
        auto swp = [](half8 v, float a, float b) {
            half8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const half2 p = half2{v[2 * e + 1], v[2 * e]} * half2{(_Float16)a, (_Float16)b};
                o[2 * e] = p[0]; o[2 * e + 1] = p[1];
            }
            return o;
        };
        // SUM: a step's three partial products are summed from zero, the small ones first, and added to the running sums by
        // vector instructions.  The matrix instruction rounds its running sum twice as coarsely as an addition does: over
        // 45 of them in a row (48 images, five taps) that is 2.1e-7 of the result, 0.6e-7 this way, for 8 % more time.
        const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
#define ZNNI_XD_MFMA(D, A, X, C) D = XROWS ? __builtin_amdgcn_mfma_f32_16x16x32_f16(X, A, C, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_f16(A, X, C, 0, 0, 0)
        if constexpr (2 * RT > CT) {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const half8 hr = xs[16 * c], lr = xs[4 * XW + 16 * c];
                const half8 hi = swp(hr, -1.f, 1.f), li = swp(lr, -1.f, 1.f);
                constexpr int RG = RT == 4 ? 2 : 3;              // row tiles at a time: enough products that do not wait for each other
#pragma unroll
                for (int r0 = 0; r0 < RT; r0 += RG) {
                    floatx4 tr[RG], ti[RG];
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { tr[r - r0] = SUM ? zero : re[r][c]; ti[r - r0] = SUM ? zero : im[r][c]; }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_XD_MFMA(tr[r - r0], ah[r], lr, tr[r - r0]); ZNNI_XD_MFMA(ti[r - r0], ah[r], li, ti[r - r0]); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_XD_MFMA(tr[r - r0], al[r], hr, tr[r - r0]); ZNNI_XD_MFMA(ti[r - r0], al[r], hi, ti[r - r0]); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) { ZNNI_XD_MFMA(tr[r - r0], ah[r], hr, tr[r - r0]); ZNNI_XD_MFMA(ti[r - r0], ah[r], hi, ti[r - r0]); }
#pragma unroll
                    for (int r = r0; r < RT && r < r0 + RG; ++r) {
                        re[r][c] = SUM ? re[r][c] + tr[r - r0] : tr[r - r0];
                        im[r][c] = SUM ? im[r][c] + ti[r - r0] : ti[r - r0];
                    }
                }
            }
        } else {
            // Few row tiles for many column tiles: the second form of an operand from the kernels' side, once a step (1 x 2 to
            // 1 x 4 tiles and 2 x 4 tiles take 1 to 2 % less of the layer, 2 -> 2 of 220 x 110 x 129, 6^3 kernels 126.6 -> 123.4 us;
            // 2 x 3 tiles took 2 % more).
            half8 bh[RT], bl[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) { bh[r] = swp(ah[r], 1.f, -1.f); bl[r] = swp(al[r], 1.f, -1.f); }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const half8 hr = xs[16 * c], lr = xs[4 * XW + 16 * c];
                floatx4 tr[RT], ti[RT];
#pragma unroll
                for (int r = 0; r < RT; ++r) { tr[r] = SUM ? zero : re[r][c]; ti[r] = SUM ? zero : im[r][c]; }
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_XD_MFMA(tr[r], ah[r], lr, tr[r]); ZNNI_XD_MFMA(ti[r], bh[r], lr, ti[r]); }
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_XD_MFMA(tr[r], al[r], hr, tr[r]); ZNNI_XD_MFMA(ti[r], bl[r], hr, ti[r]); }
#pragma unroll
                for (int r = 0; r < RT; ++r) { ZNNI_XD_MFMA(tr[r], ah[r], hr, tr[r]); ZNNI_XD_MFMA(ti[r], bh[r], hr, ti[r]); }
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    re[r][c] = SUM ? re[r][c] + tr[r] : tr[r];
                    im[r][c] = SUM ? im[r][c] + ti[r] : ti[r];
                }
            }
        }
#undef ZNNI_XD_MFMA
    };
    // A pair's kernel operands are parked while the pair before it is multiplied, into the half that was read before that.
    if (EARLY && live) request();                            // (the first chunk's rows and kernel operands travel together)
    if (t < RT * 16) rjs[t] = g.rinv[mblk * RT * 16 + t];
    park_a(0, 0);
    if (nsteps > 2) load_a();
    const half8* const as0 = As + kk * RT * 32 + l16;
    for (int gs = 0, buf = 0; gs < nsteps; gs += 2, buf ^= 1) {
        // this pair's operands are in place, the last one's are free (staged together, the first chunk's barriers say so)
        if (!SHARED || gs) __syncthreads();
        if (live) step(as0 + buf * RT * 256);
        if (gs + 2 < nsteps) {
            park_a(gs + 2, buf ^ 1);
            if (gs + 4 < nsteps) load_a();
        }
        if (live && gs + 1 < nsteps) step(as0 + buf * RT * 256 + RT * 128);
    }
    if (!live) return;

    // Kernels of an output image of uneven size: every image counts by itself, next to the largest value of all.  (Read again for
    // it: looking at them one by one as they are staged took 6 to 11 % of the kernel where images are few, with even kernels too:
    // 2 x 3 -> 1 of 142 x 178 x 255, 3^3 206 us, 186 this way, 185 without any check.)
    // (the lane's number anew: kept from the start, it takes a register that three by two tiles have to spill)
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
        const float2* const a1 = g.A1 + (size_t)poz * g.ky * per + mblk * RT * 16 + l16;
        auto again = [&](int r, int i, int tap) {
            float2 s = make_float2(0.f, 0.f);
            for (int b = 0, t = 0; b < g.ky; ++b) {          // t = (poy * b) mod Ny
                s = cfma(s, a1[b * per + ((size_t)tap * g.fp + i) * g.Mp + r * 16], g.tw[t]);
                t += poy;
                if (t >= g.Ny) t -= g.Ny;
            }
            const float cr = g.row[(mblk * RT + r) * 16 + l16] * g.scale, ci = g.cinv[i];
            return make_float2(s.x * cr * ci, s.y * cr * ci);
        };
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) { re[r][c] = floatx4{0.f, 0.f, 0.f, 0.f}; im[r][c] = re[r][c]; }
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
                    const half2 ah = reinterpret_cast<const half2*>(ap + r * 32)[q], al = reinterpret_cast<const half2*>(ap + r * 32 + 16)[q];
                    float ar = (float)ah[0] + (float)al[0], ai = (float)ah[1] + (float)al[1];
                    if (uneven) { const float2 e = again(r, 4 * qd + q, tap); ar = e.x; ai = e.y; }
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        auto mm = [](float p, float v, floatx4& d) {
                            d = XROWS ? __builtin_amdgcn_mfma_f32_16x16x4f32(v, p, d, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x4f32(p, v, d, 0, 0, 0);
                        };
                        mm(ar, x[c].x, re[r][c]);
                        mm(ar, x[c].y, im[r][c]);
                        mm(ai, -x[c].y, re[r][c]);
                        mm(ai, x[c].x, im[r][c]);
                    }
                }
            }
        }
    }

    // ---- results.  The smaller factor first: either alone may be out of range where the result is not.  Rows of Yd are
    // padded to whole fours.
    const float inv = pow2f(-sexp);
    auto scale_of = [&](int row) { return __uint_as_float(__float_as_uint(rjs[row]) & 0x7f800000u); };
    float2* const ypen = g.Yd + (size_t)poz * g.ypen + (size_t)poy * g.yrow;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int j0 = (mblk * RT + r) * 16;
        if constexpr (XROWS) {                               // element e of lane (kk, l16): image l16, output 4 kk + e
            if (j0 + l16 >= g.fo) continue;
            const float s = scale_of(r * 16 + l16), f0 = fminf(inv, s), f1 = fmaxf(inv, s);
            float2* y = ypen + (size_t)(unsigned)(sI * g.fo + j0 + l16) * g.yimg;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int xo = col0 + c * 16 + 4 * kk;
                if (xo >= g.nox) continue;
                float4* d = reinterpret_cast<float4*>(y + xo);
                float4 v0 = make_float4(re[r][c][0] * f0 * f1, im[r][c][0] * f0 * f1, re[r][c][1] * f0 * f1, im[r][c][1] * f0 * f1);
                float4 v1 = make_float4(re[r][c][2] * f0 * f1, im[r][c][2] * f0 * f1, re[r][c][3] * f0 * f1, im[r][c][3] * f0 * f1);
                if (g.accumulate) {
                    const float4 o0 = d[0], o1 = d[1];
                    v0.x += o0.x; v0.y += o0.y; v0.z += o0.z; v0.w += o0.w;
                    v1.x += o1.x; v1.y += o1.y; v1.z += o1.z; v1.w += o1.w;
                }
                d[0] = v0;
                d[1] = v1;
            }
        } else {                                             // ... image 4 kk + e, output l16
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = j0 + 4 * kk + e;
                if (j >= g.fo) break;
                const float s = scale_of(r * 16 + 4 * kk + e), f0 = fminf(inv, s), f1 = fmaxf(inv, s);
                float2* y = ypen + (size_t)(unsigned)(sI * g.fo + j) * g.yimg;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const int xo = col0 + c * 16 + l16;
                    if (xo >= g.nox) continue;
                    float2* d = y + ((xo >> 2) * g.yblk + (xo & 3));
                    float2 v = make_float2(re[r][c][e] * f0 * f1, im[r][c][e] * f0 * f1);
                    if (g.accumulate) { const float2 o = *d; v.x += o.x; v.y += o.y; }
                    *d = v;
                }
            }
        }
    }
}

// Rows of X2 and Yd along x.
template <int RT, int CT, bool SUM>
__global__ __launch_bounds__(256, (xd_blocks<RT, CT, false>())) void k_mac_xd(XdArgs g)
{
    extern __shared__ half8 lds[];
    xd_body<RT, CT, SUM, false>(g, lds);
}
// Rows in blocks of four x, a block of every oy after the other, as the kernels of passes_fused.hip that take four planes
// leave and read them.  Four neighbouring pencils share every cache line: they are neighbours on one XCD.
template <int RT, int CT>
__global__ __launch_bounds__(256, (xd_blocks<RT, CT, true>())) void k_mac_planes(XdArgs g)
{
    extern __shared__ half8 lds[];
    xd_body<RT, CT, true, true>(g, lds);
}

// ---------------------------------------------------------------------------------------- kernel transform
// Second stage (y) of the kernel transform for this route: A1 (after the z stage) -> the split operand layout above,
//     A[pencil][slot][j / 16][hi, lo][j % 16][image of the quad][re, im] = split( rs[j] * scale *
//         sum_{b<ky} A1[oz][b][a][i][j] exp(-2 pi i oy b / Ny) ),
// slots of a pencil in the order the contraction walks them: chunks of four image quads, inside a chunk tap by tap,
// quads fastest.  One thread: one (slot, j), whose four images' ky values it keeps in registers while it walks KX_OY
// bins along y; 16 + 16 bytes per bin leave it, 256 contiguous bytes per sixteen threads.  Bound by writing A.
// (noy = KX_OY bins, or fewer where that leaves the chip short of workgroups)
constexpr int KX_OY = 32;
__device__ __forceinline__ void xd_store(half8* d, const float2 (&v)[4])
{
    half8 h, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        _Float16 x, y;
        split2(v[q].x, 1.f, x, y);
        h[2 * q] = x; l[2 * q] = y;
        split2(v[q].y, 1.f, x, y);
        h[2 * q + 1] = x; l[2 * q + 1] = y;
    }
    d[0] = h;
    d[16] = l;
}
template <int KY>          // taps along y; 0: any number, A1 read again for every bin
__global__ __launch_bounds__(256) void k_kprep_xd(const float2* __restrict__ A1, half8* __restrict__ A,
                                                  const float2* __restrict__ tw, const float* __restrict__ rs,
                                                  const float* __restrict__ cinv, int N, int ky, int K, int fp, int Mp, float scale, int noy)
{
    constexpr int KT = KY ? KY : 1;
    __shared__ float2 tw2[KX_OY][KT];
    const int idx = blockIdx.x * 256 + threadIdx.x;
    const int oy0 = blockIdx.y * noy, oz = blockIdx.z;
    const int fq = fp >> 2, nslots = K * fq;
    if constexpr (KY) {
        for (int e = threadIdx.x; e < noy * KY; e += 256) {
            const int o = e / KT, b = e - o * KT;
            tw2[o][b] = tw[(unsigned)((oy0 + o) * b) % (unsigned)N];
        }
        __syncthreads();
    }
    if (idx >= nslots * Mp) return;
    const int j = idx % Mp, slot = idx / Mp;
    int quad, a;
    xd_slot(slot, K, fq, quad, a);
    const size_t per = (size_t)K * fp * Mp;
    const float2* a1 = A1 + (size_t)oz * ky * per + ((size_t)a * fp + 4 * quad) * Mp + j;
    const float s = rs[j] * scale;                       // scale is no power of two: folded in before the split
    float ci[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) ci[q] = cinv[4 * quad + q];
    const int no = min(noy, N - oy0);
    half8* d = A + ((size_t)(oz * N + oy0) * nslots + slot) * 2 * Mp + (j >> 4) * 32 + (j & 15);
    const size_t dstep = (size_t)nslots * 2 * Mp;
    if constexpr (KY) {
        float2 v[KT][4];
#pragma unroll
        for (int b = 0; b < KT; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float2 x = a1[(size_t)b * per + q * Mp];
                v[b][q] = make_float2(x.x * s * ci[q], x.y * s * ci[q]);
            }
        for (int o = 0; o < no; ++o, d += dstep) {
            float2 acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[q] = make_float2(0.f, 0.f);
#pragma unroll
                for (int b = 0; b < KT; ++b) acc[q] = cfma(acc[q], v[b][q], tw2[o][b]);
            }
            xd_store(d, acc);
        }
    } else {
        for (int o = 0; o < no; ++o, d += dstep) {
            float2 acc[4] = {};
            int t = 0;                                   // (oy * b) mod N
            for (int b = 0; b < ky; ++b) {
                const float2 w = tw[t];
                t += oy0 + o;
                if (t >= N) t -= N;
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = cfma(acc[q], a1[(size_t)b * per + q * Mp], w);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = make_float2(acc[q].x * s * ci[q], acc[q].y * s * ci[q]);
            xd_store(d, acc);
        }
    }
}

template <int KY>
static znni_status launch_kprep_xd_k(const LayerPlan& L, hipStream_t st)
{
    const Dims& d = L.d;
    const int items = d.kx * (L.fp >> 2) * L.Mp;
    const int nb = (items + 255) / 256;
    int noy = KX_OY;
    while (noy > 4 && (long long)nb * ((d.Ny + noy - 1) / noy) * L.ozn < 1024) noy >>= 1;
    k_kprep_xd<KY><<<dim3(nb, (d.Ny + noy - 1) / noy, L.ozn), dim3(256), 0, st>>>(
        L.A1 + (size_t)L.oz0 * d.ky * d.kx * L.fp * L.Mp, reinterpret_cast<half8*>(L.A), L.twy, split_scales(L).row, split_scales(L).cinv, d.Ny, d.ky, d.kx, L.fp, L.Mp, xd_scale(d), noy);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    return ZNNI_OK;
}

znni_status launch_kprep_xd(const LayerPlan& L, hipStream_t st)
{
    switch (L.d.ky) {
        case 1: return launch_kprep_xd_k<1>(L, st);
        case 2: return launch_kprep_xd_k<2>(L, st);
        case 3: return launch_kprep_xd_k<3>(L, st);
        case 4: return launch_kprep_xd_k<4>(L, st);
        case 5: return launch_kprep_xd_k<5>(L, st);
        case 6: return launch_kprep_xd_k<6>(L, st);
        case 7: return launch_kprep_xd_k<7>(L, st);
        case 8: return launch_kprep_xd_k<8>(L, st);
        case 9: return launch_kprep_xd_k<9>(L, st);
    }
    return launch_kprep_xd_k<0>(L, st);
}

// ---------------------------------------------------------------------------------------- host side
// Widest strip of a wave for a row block (its sums take RT * CT * 8 registers a lane and have to leave room for two waves
// per SIMD).
template <int RT> constexpr int xd_max_ct() { return RT >= 4 ? 3 : 5; }
bool mac_xd_available(const LayerPlan& L) { return L.d.kx >= 1 && L.d.kx <= XD_MAX_K; }

static XdArgs xd_args(const LayerPlan& L, int accumulate)
{
    const Dims& d = L.d;
    XdArgs g;
    g.A = reinterpret_cast<const half8*>(L.A); g.rinv = split_scales(L).rinv;
    g.A1 = L.A1 + (size_t)L.oz0 * d.ky * d.kx * L.fp * L.Mp; g.row = split_scales(L).row; g.cinv = split_scales(L).cinv;
    g.tw = L.twy; g.scale = xd_scale(d); g.ky = d.ky; g.fp = L.fp;
    const int rows = L.tiles ? d.Nz : L.ozn;
    g.zc = L.tiles ? d.zc : rows; g.Nz = d.Nz;
    if (L.planes) {
        const unsigned nb = (unsigned)(d.nx + 3) / 4, nbo = (unsigned)(d.nox + 3) / 4, zr = L.tiles ? d.Nz : d.zc;
        g.xpen = (size_t)nb * d.Ny * 4; g.ximg = zr * (unsigned)g.xpen; g.xrow = 4; g.xblk = d.Ny * 4;
        g.ypen = (size_t)nbo * d.Ny * 4; g.yimg = zr * (unsigned)g.ypen; g.yrow = 4; g.yblk = d.Ny * 4;
    } else {
        g.ximg = (unsigned)d.x2i * (unsigned)d.ldx; g.xpen = (size_t)d.x2o * d.ldx; g.xrow = d.ldx; g.xblk = 4;
        g.yimg = (unsigned)d.ydi * (unsigned)d.ldxo; g.ypen = (size_t)d.ydo * d.ldxo; g.yrow = d.ldxo; g.yblk = 4;
    }
    g.f = L.f; g.fo = L.fo; g.Mp = L.Mp; g.K = d.kx;
    g.nx = d.nx; g.nox = d.nox; g.Ny = d.Ny;
    g.npencils = rows * d.Ny; g.accumulate = accumulate;
    g.X2 = L.buf1 + (size_t)L.oz0 * g.xpen; g.Yd = L.Yt + (size_t)L.oz0 * g.ypen;
    return g;
}

template <int RT, int CT, bool SUM, bool PLANES>
static znni_status launch_xd(const LayerPlan& L, int accumulate, hipStream_t st)
{
    const Dims& d = L.d;
    XdArgs g = xd_args(L, accumulate);
    constexpr int PER = xd_shared(RT, CT, PLANES) ? 4 : 1;        // strips that are staged together and count as one here
    const int spr = ((d.nox + 15) / 16 + CT * PER - 1) / (CT * PER), pg = PLANES ? 4 : 1;
    g.nstrips = L.S * spr;
    const int nwg = (g.nstrips * PER + 3) / 4, nsub = nwg * L.mac_nmblk;
    g.d_sub.set((unsigned)(nsub * pg)); g.d_pg.set((unsigned)pg); g.d_spr.set((unsigned)spr); g.d_nwg.set((unsigned)nwg);
    g.d_Ny.set((unsigned)d.Ny);
    const long long blocks = (long long)((g.npencils + 8 * pg - 1) / (8 * pg)) * nsub * pg * 8;
    if (blocks > 0x7fffffffll) return ZNNI_ERR_SHAPE;
    constexpr size_t lds = xd_lds_bytes<RT, CT, PLANES>();
    void (*kernel)(XdArgs);
    if constexpr (PLANES) kernel = k_mac_planes<RT, CT>;
    else kernel = k_mac_xd<RT, CT, SUM>;
    if (lds > 48 * 1024 && hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return ZNNI_ERR_HIP;
    kernel<<<dim3((unsigned)blocks), dim3(256), lds, st>>>(g);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    return ZNNI_OK;
}

// Columns: the strip width whose waves, dealt four to a workgroup, are through a chunk first: its products, its rounds of
// staging and what a wave waits for in any case (in cycles of a SIMD; products 16 per matrix instruction, 200 per round, 800).
// Of two that tie the wider one.  Fewer waves than the chip has SIMDs all run at once, so that only the time of one counts (without
// that: 5 x 613 -> 26 of 7 x 7 x 10, 2^3 kernels 164 us for the layer, 141 with it; 2 x 306 -> 80 of 15 x 9 x 13,
// 5^3 219 and 200).
template <int RT, bool SUM, bool PLANES>
static znni_status launch_xd_cols_s(const LayerPlan& L, int accumulate, hipStream_t st)
{
    constexpr int MAXCT = xd_max_ct<RT>();
    constexpr long long FULL = 1024;                         // (of the whole layer: its slabs take the same width)
    const int tiles = (L.d.nox + 15) / 16;
    int CT = 1;
    long long best = -1;
    for (int c = 1; c <= MAXCT; ++c) {
        const int PER = xd_shared(RT, c, PLANES) ? 4 : 1;
        const long long waves = ((long long)L.S * ((tiles + c * PER - 1) / (c * PER)) * PER + 3) / 4 * 4;
        const int rounds = (4 * (16 * c + 8) + 63) / 64;
        const long long n = std::max(waves * L.d.zc * L.d.Ny * L.mac_nmblk, FULL) * (96 * L.d.kx * RT * c + 200 * rounds + 800);
        if (best < 0 || n <= best) { best = n; CT = c; }
    }
    switch (CT) {
        case 1: return launch_xd<RT, 1, SUM, PLANES>(L, accumulate, st);
        case 2: return launch_xd<RT, 2, SUM, PLANES>(L, accumulate, st);
        case 3: return launch_xd<RT, 3, SUM, PLANES>(L, accumulate, st);
        case 4: if constexpr (MAXCT >= 4) return launch_xd<RT, 4, SUM, PLANES>(L, accumulate, st); break;
        case 5: if constexpr (MAXCT >= 5) return launch_xd<RT, 5, SUM, PLANES>(L, accumulate, st); break;
    }
    return ZNNI_ERR_SHAPE;
}

// Stepwise sums wherever another form of the multiply-accumulate, which the call could have taken, would be closer to
// the 64-bit result without them: the block form (four and five taps, at least 16 images: sums a fifth as long; 48 -> 48
// images of 320^2, 5^3 kernels: 3.3e-7 off without stepwise sums, 2.45e-7 with them, 3.0e-7 in blocks) and the batch form.
// It is no rule on the length of the sums: with seven taps and 80 images they are longer, but the fp32 products this
// kernel replaced there were at 5.4e-7 against its 3.7e-7, and stepwise sums cost 8 % of the kernel.
template <int RT>
static znni_status launch_xd_cols(const LayerPlan& L, int accumulate, hipStream_t st)
{
    if (L.planes) return launch_xd_cols_s<RT, true, true>(L, accumulate, st);
    return mac_xb_available(L) || mac_batch_preferred(L) ? launch_xd_cols_s<RT, true, false>(L, accumulate, st)
                                                         : launch_xd_cols_s<RT, false, false>(L, accumulate, st);
}

znni_status launch_mac_xd(const LayerPlan& L, int accumulate, hipStream_t st)
{
    if (!mac_xd_available(L)) return ZNNI_ERR_UNSUPPORTED_SIZE;
    if (L.tiles) return accumulate ? ZNNI_ERR_SHAPE : launch_mac_quads(L, xd_args(L, 0), st);     // (sub-layers go through whole planes)
    switch (L.mac_RTW) {
        case 1: return launch_xd_cols<1>(L, accumulate, st);
        case 2: return launch_xd_cols<2>(L, accumulate, st);
        case 3: return launch_xd_cols<3>(L, accumulate, st);
        case 4: return launch_xd_cols<4>(L, accumulate, st);
        case 5: return launch_xd_cols<5>(L, accumulate, st);
    }
    return ZNNI_ERR_SHAPE;
}

}  // namespace znni
