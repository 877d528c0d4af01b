// passes_fused.hip -- the transforms along y and z in one kernel, for images whose (oz, oy) plane fits LDS.
//
// Inverse side:
// When the transform lengths along y and z are equal and at most about 120, the plane Y2[imgo][.][xo][.] of one
// (output image, xo) -- zc rows of N complex values, 58 KB at N = 120 -- fits the 160 KB of LDS of a CU more than
// once.  One workgroup then does what the separate inverse y and inverse z passes do (Section III-B/C, the last
// two steps of the inverse transform, pruned to the valid outputs, with bias and transfer function,
// Section IV-A-3) without the intermediate tensor Y1 going to HBM and back: it reads the plane's rows as they
// lie, inverse-transforms them along y keeping the valid yo in LDS, then takes pairs of yo columns through the
// complex-to-real inverse along z and writes the (yo, zo) plane of the output image, which is contiguous.  Per
// output image that moves 8 N zc nox + 4 nox noy noz bytes instead of that plus 16 zc nox noy.
//
// Forward side, the mirror image: one workgroup reads the (y, z) plane of one (input image, x) -- contiguous in
// the input tensor --, transforms pairs of rows real-to-complex along z into LDS, then every oz column along y, and
// writes X2'[img][x][oz][oy] as whole rows; the intermediate tensor X1 never exists.  The forward x pass that
// follows reads X2' with a transposing load (P_FWD_XT in passes_fast.hip).
//
// Every line is transformed by the same two in-register steps as in passes_fast.hip (two_step.h), all lines of the
// plane in one round (one thread per (line, sample offset); zc lines, or N / 2 where the two real ones ride as one,
// see the kernels).  The exchange buffer of the two steps, the plane between the two transforms (inverse) and the
// raw input plane (forward) take turns in ONE region of zc x (N + 2) complex values: whatever is read next sits in
// registers across the barrier that hands the region over.  That is 42 KB at N = 100 -- three workgroups per CU,
// where separate regions (83 KB) left room for one, and a workgroup's life is a chain of memory round trips and
// barriers that only other workgroups can fill.  The forward kernel exists up to length 128, the inverse up to 120.
//
// Both also exist for four neighbouring x of layers whose x axis is not transformed (k_fwd_zy_planes, k_inv_yz_planes, up to
// length 64).
#include <algorithm>
#include "kprep.h"
#include "two_step.h"

namespace znni {

struct FusedArgs {
    const float2* src;     // Y2[imgo][oz][xo][oy]
    float* out;
    const float2* tw;      // [N]
    const float* bias;
    Dims d;
    int fo, relu;
    int QP;                // pitch of the plane kept in LDS (noy + 1 or + 2, even)
};

// Threads of a workgroup, and the number of waves per SIMD the register allocation is held to.  By default four
// (128 registers); the listed kernels sit a few registers above the step that lets one more workgroup share the
// CU and are held below it.
template <int R1, int R2>
constexpr int fused_nth() { return ((R1 * R2 / 2 + 1) * (R1 > R2 ? R1 : R2) + 63) / 64 * 64; }
// The forward kernel can do with N / 2 lines per direction instead of N / 2 + 1 (see there).  It does where that
// saves a wave per workgroup and was measured faster (7 to 21 % at 32, 48, 64; 2 % at 96) and at 128, which then fits
// one round of 1024 threads; where no wave is saved the special cases cost up to 10 % (24), and at 112 it was 5 %
// slower in spite of the wave saved.
constexpr bool fused_fwd_packs(int N) { return N == 32 || N == 48 || N == 64 || N == 96 || N == 128; }
template <int R1, int R2>
constexpr int fused_nth_fwd()
{
    return ((R1 * R2 / 2 + (fused_fwd_packs(R1 * R2) ? 0 : 1)) * (R1 > R2 ? R1 : R2) + 63) / 64 * 64;
}
template <int R1, int R2, bool FWD>
constexpr int fused_waves()
{
    constexpr int N = R1 * R2;
    // measured (32 -> 32 images, batches of 1.5 GB): inverse at 96 held to 64 registers (two over; three workgroups
    // per CU instead of two) 14 % faster, inverse at 112 3-4 %; where the step is further away the spills cost 5 to
    // 25 %.  (The forward kernels need no budget: since they untangle on the way into the y transform they use 38
    // to 68 registers.)
    if (!FWD && (N == 96 || N == 112)) return 8;
    // forward at 128: 1024 threads; at 76 registers one workgroup has a CU to itself, held to 64 (16 bytes of
    // scratch) two share it: 0.24 -> 0.19 ms for 40 images of 128^3
    if (FWD && N == 128) return 8;
    return 4;
}

// The inverse kernel can pack the same two lines: rows oz = 0 and N / 2 of the plane are spectra of real sequences,
// so c = row 0 + i row N/2 comes back from the inverse y transform as (row 0's values, row N/2's values).  Measured:
// 11-12 % faster at 32 and 64 (a wave less per workgroup), a tie at 48, 3 % slower at 96; at 128 the kernel it makes
// possible (1024 threads, held to 64 registers with 36 bytes of scratch) is 13 % slower than the two separate
// passes on 40 images of 128^3 and 16-19 % faster on 32 or 8 images: not used there.
constexpr bool fused_inv_packs(int N) { return N == 32 || N == 64; }
template <int R1, int R2>
constexpr int fused_nth_inv()
{
    return ((R1 * R2 / 2 + (fused_inv_packs(R1 * R2) ? 0 : 1)) * (R1 > R2 ? R1 : R2) + 63) / 64 * 64;
}

constexpr int PLANES = 4, PLANES_MAX = 64;    // (above length 64 four planes at once would be over 1024 threads)

// NP planes from the samples v of their y lines (conjugated, as the loads leave them) to the rows of the output images,
// plane p at dst + p * pitch.  Of NP neighbouring threads each works on another plane.  R: per plane, RS elements apart,
// [ZC][P] exchange buffer; between the transforms the plane Q[ZC][QP].  nplanes: planes of a
// block of four that exist from the first of these on.
template <int R1, int R2, int NP>
__device__ __forceinline__ void inv_plane(float2 (&v)[R1], const float2* tws, float2* const R0, int RS, int QP, const Dims& d,
                                          float* dst0, size_t pitch, int nplanes, float bj, int relu)
{
    using TS = TwoStep<R1, R2>;
    constexpr int N = TS::N, P = TS::P, ZC = N / 2 + 1;
    constexpr bool PACK = fused_inv_packs(N);
    constexpr int NL = PACK ? N / 2 : ZC;     // lines per transform
    const int t = threadIdx.x / NP, NTH = blockDim.x / NP;
    float2* const R = R0 + threadIdx.x % NP * RS;
    const int noy = d.noy, noz = d.noz;
    const int ja = t % R2, la = t / R2;       // step A: (line la, sample offset ja)
    const bool in_a = la < NL;
    const int lb = t % NL, q = t / NL;        // step B: (line lb, output offset q); work only for q < R1
    float2 u[R2];

    if (in_a) TS::step_a(v, la, ja, tws, R);
    __syncthreads();
    if (q < R1) TS::step_b(u, lb, q, R);
    __syncthreads();                          // the exchange buffer has been read: the region becomes Q
    if (q < R1) {
#pragma unroll
        for (int r = 0; r < R2; ++r) {
            const int yo = q + R1 * r - (d.ky - 1);
            if (yo >= 0 && yo < noy) {
                if (!PACK || lb) {
                    R[lb * QP + yo] = cconj(u[r]);
                } else {                      // real part: row 0, imaginary part of the conjugate: row N/2
                    R[yo] = make_float2(u[r].x, 0.f);
                    R[(N / 2) * QP + yo] = make_float2(-u[r].y, 0.f);
                }
            }
        }
    }
    {
        const int sh = QP - noy - 1;                         // one or two spare columns, read by the last yo pair
        for (int e = t; e < (ZC << sh); e += NTH) R[(e >> sh) * QP + noy + (e & sh)] = make_float2(0.f, 0.f);
    }
    __syncthreads();

    // ---- inverse along z, complex to real: yo columns 2p and 2p+1 ride as real and imaginary part of one line
    const int np = (noy + 1) >> 1;            // <= N / 2 < ZC lines
    if (in_a) {
        const float mp = la < np ? 1.f : 0.f;
        const float2* col = R + 2 * min(la, np - 1);
#pragma unroll
        for (int m = 0; m < R1; ++m) {
            const int e = ja + R2 * m;
            const bool direct = e < ZC;
            const int ee = direct ? e : N - e;
            const float4 ab = *reinterpret_cast<const float4*>(col + ee * QP);
            float2 A = make_float2(ab.x * mp, ab.y * mp), B = make_float2(ab.z * mp, ab.w * mp);
            if (!direct) { A = cconj(A); B = cconj(B); }
            v[m] = cconj(cadd(A, mul_pi(B)));
        }
    }
    __syncthreads();                          // Q has been read: the region is the exchange buffer again
    if (in_a) TS::step_a(v, la, ja, tws, R);
    __syncthreads();
    if (q < R1) TS::step_b(u, lb, q, R);
    __syncthreads();
    if (q < R1) {
#pragma unroll
        for (int r = 0; r < R2; ++r) R[lb * P + q + R1 * r] = u[r];           // natural order per line
    }
    __syncthreads();
    // rows yo of out[imgo][xo]: real part of line l -> row 2l, minus imaginary part -> row 2l+1
    // a wave per line = pair of rows (one LDS read serves both), or per two or four lines where rows are at most 32
    // or 16 long
    constexpr int LW = N <= 16 ? 16 : N <= 32 ? 32 : 64, RPI = 64 / LW;
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64, nw = blockDim.x / 64;
    for (int i = w * RPI + lane / LW; i < np * NP; i += nw * RPI) {
        const int l = i / NP, p = i % NP;
        if (NP > 1 && p * (PLANES / NP) >= nplanes) continue;
        const float2* row = R0 + p * RS + l * P + (d.kz - 1);
        float* d0 = dst0 + p * pitch + (size_t)(2 * l) * noz;
        const bool two = 2 * l + 1 < noy;
        for (int zo = lane % LW; zo < noz; zo += LW) {
            const float2 c = row[zo];
            float v0 = c.x + bj, v1 = bj - c.y;
            if (relu) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); }
            d0[zo] = v0;
            if (two) d0[noz + zo] = v1;
        }
    }
}

template <int R1, int R2>
__global__ __launch_bounds__((fused_nth_inv<R1, R2>())) __attribute__((amdgpu_waves_per_eu((fused_waves<R1, R2, false>()))))
void k_inv_yz(FusedArgs a)
{
    using TS = TwoStep<R1, R2>;
    constexpr int N = TS::N, ZC = N / 2 + 1;
    constexpr bool PACK = fused_inv_packs(N);
    constexpr int NL = PACK ? N / 2 : ZC;     // lines per transform
    extern __shared__ float2 lds[];
    float2* tws = lds;                 // [N]
    const int t = threadIdx.x, NTH = blockDim.x;
    const int xo = blockIdx.x, img = blockIdx.y;
    const Dims& d = a.d;
    const int nox = d.nox;

    for (int q = t; q < N; q += NTH) tws[q] = a.tw[q];

    const int ja = t % R2, la = t / R2;       // step A: (line la, sample offset ja)
    const bool in_a = la < NL;
    float2 v[R1];

    // ---- inverse along y: the rows oz of the plane, conj . forward . conj
    if (in_a) {
        const float2* row = a.src + (((size_t)img * ZC + la) * nox + xo) * d.ldn;
        if (!PACK || la) {
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const float2 x = row[ja + R2 * m];
                v[m] = make_float2(x.x, -x.y);
            }
        } else {                              // line 0 = row 0 + i row N/2, conjugated
            const float2* rown = row + (size_t)(N / 2) * nox * d.ldn;
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const float2 x = row[ja + R2 * m], y = rown[ja + R2 * m];
                v[m] = make_float2(x.x - y.y, -(x.y + y.x));
            }
        }
    }
    __syncthreads();                          // twiddles are in LDS
    inv_plane<R1, R2, 1>(v, tws, lds + N, 0, a.QP, d, a.out + (((size_t)img * nox + xo) * d.noy) * d.noz, 0, 1,
                         a.bias ? a.bias[img % a.fo] : 0.f, a.relu);
}

// Four neighbouring x at a time, for layers whose x axis is not transformed (mac_xd.hip): their spectra lie as
// [img][oz][x / 4][oy][x % 4], so that the multiply-accumulate, which reads rows along x, finds 32 bytes together, and a row
// of a workgroup's blocks is one run.  A workgroup either takes all four planes at once, of four neighbouring threads each
// works on another one, or one plane after the other, a thread's values of all four in registers.  (Two at a time is slower
// than either, and so is storing or loading fewer than the 32 bytes: 8 at a time three times, 16 at a time 1.5 times.)
// Together where the lines of a plane fill whole waves (or a fraction of one), one by one elsewhere: workgroups of 11 to 15
// waves leave a CU to two of them that wait at the same barriers.  Measured, together against one by one, us: forward at
// 64 (8 x 32 images) 108, 141; 56 (64 x 80 of 51^3) 1851, 1521; 48 238, 258; 40 103, 90; 32 58, 65; 20 60, 55; 14 49, 67.
// Inverse at 64 107, 122; 56 1795, 1564; 48 311, 250; 40 115, 88; 32 239, 224; 20 49, 48; 14 33, 40.
// Where there are too few workgroups to fill the chip four planes one by one are four times the latency: always together.
constexpr bool planes_wide(int N, bool packs) { return packs || N <= 14; }
constexpr long long PLANES_FEW = 1024;
constexpr int planes_nth(int lines, int T, int par) { return (par * lines * T + 63) / 64 * 64; }
// elements from one plane's region to the next: whole rows of the 64 banks and a quarter
constexpr int planes_pitch(int region) { return (region + 31) / 32 * 32 + 8; }
template <int R1, int R2, int PAR_, bool FWD>
struct Planes {
    static constexpr int N = R1 * R2;
    static constexpr bool PACK = FWD ? fused_fwd_packs(N) : fused_inv_packs(N);
    static constexpr int NL = N / 2 + (PACK ? 0 : 1);                   // lines per transform
    static constexpr int PAR = PAR_, ROUNDS = PLANES / PAR;
    static constexpr int NTH = planes_nth(NL, R1 > R2 ? R1 : R2, PAR);
    static constexpr int RS = planes_pitch((FWD ? NL : N / 2 + 1) * (N + 2));
    // registers: one by one, three (forward) or four waves per SIMD
    static constexpr int WAVES = PAR > 1 ? 4 : FWD ? 3 : 4;
};

template <int R1, int R2, int PAR_>
__global__ __launch_bounds__((Planes<R1, R2, PAR_, false>::NTH)) __attribute__((amdgpu_waves_per_eu((Planes<R1, R2, PAR_, false>::WAVES))))
void k_inv_yz_planes(FusedArgs a)
{
    using PL = Planes<R1, R2, PAR_, false>;
    constexpr int N = PL::N, ZC = N / 2 + 1, PAR = PL::PAR, ROUNDS = PL::ROUNDS;
    extern __shared__ float2 lds[];
    float2* tws = lds;
    const int t = threadIdx.x / PAR, p = threadIdx.x % PAR;
    const int xb = blockIdx.x, img = blockIdx.y, nxb = gridDim.x;
    const Dims& d = a.d;

    for (int q = threadIdx.x; q < N; q += blockDim.x) tws[q] = a.tw[q];

    const int ja = t % R2, la = t / R2;
    // this thread's values of the ROUNDS planes p * ROUNDS + h
    struct alignas(8 * (ROUNDS > 1 ? 2 : 1)) Run { float2 v[ROUNDS]; };
    float2 v[ROUNDS][R1];
    if (la < PL::NL) {
        const float2* row = a.src + ((((size_t)img * ZC + la) * nxb + xb) * N + ja) * PLANES + p * ROUNDS;
        if (!PL::PACK || la) {
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const Run x = *reinterpret_cast<const Run*>(row + R2 * m * PLANES);
#pragma unroll
                for (int h = 0; h < ROUNDS; ++h) v[h][m] = make_float2(x.v[h].x, -x.v[h].y);
            }
        } else {                              // line 0 = row 0 + i row N/2, conjugated
            const float2* rown = row + (size_t)(N / 2) * nxb * N * PLANES;
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const Run x = *reinterpret_cast<const Run*>(row + R2 * m * PLANES), y = *reinterpret_cast<const Run*>(rown + R2 * m * PLANES);
#pragma unroll
                for (int h = 0; h < ROUNDS; ++h) v[h][m] = make_float2(x.v[h].x - y.v[h].y, -(x.v[h].y + y.v[h].x));
            }
        }
    }
    const size_t pitch = (size_t)d.noy * d.noz;
    const float bj = a.bias ? a.bias[img % a.fo] : 0.f;
    const int left = d.nox - PLANES * xb;                     // planes from this block's first on
#pragma unroll
    for (int h = 0; h < ROUNDS; ++h) {
        if (h >= left) break;
        __syncthreads();                      // twiddles are in LDS; the plane before has been stored
        inv_plane<R1, R2, PAR>(v[h], tws, lds + N, PL::RS, a.QP, d, a.out + ((size_t)img * d.nox + PLANES * xb + h) * pitch,
                               ROUNDS * pitch, left, bj, a.relu);
    }
}

struct FusedFwdArgs {
    const float* in;       // [img][x][y][z]
    float2* dst;           // X2'[img][x][oz][oy]
    const float2* tw;      // [N]
    Dims d;
    const float* col;      // powers of two of the f input images of a tuple (mac_xd.hip)
    int f;
    // small layers: the workgroups behind those of the images (prep_small); null: none
    const float* w;
    float2 *A1, *twx, *twz;
    SplitScales S;
    int nimg, fo, fp, Mp;
    float scale;
};

// Lines per transform: along z two real rows ride in one complex line, N / 2 lines at most.  Along y the plane has
// N / 2 + 1 lines (oz = 0 ... N / 2), but the first and the last are real sequences (sums and alternating sums of
// real rows): with PACK they ride together as real and imaginary part of line 0 and are separated, by the same
// symmetry, when the rows are stored -- N / 2 lines in both directions.
// NP raw planes [ny][nz] in R, RS elements apart (behind a barrier), to their transformed lines [NL][P] in R, in natural
// order, behind a barrier.  Of NP neighbouring threads each works on another plane.
template <int R1, int R2, int NP>
__device__ __forceinline__ void fwd_plane(const float2* tws, float2* const R0, int RS, int ny, int nz)
{
    using TS = TwoStep<R1, R2>;
    constexpr int N = TS::N, P = TS::P, ZC = N / 2 + 1;
    constexpr bool PACK = fused_fwd_packs(N);
    constexpr int NL = PACK ? N / 2 : ZC;
    const int t = threadIdx.x / NP;
    float2* const R = R0 + threadIdx.x % NP * RS;
    const int ja = t % R2, la = t / R2;
    const bool in_a = la < NL;
    const int lb = t % NL, q = t / NL;
    const float* raw = reinterpret_cast<const float*>(R);
    float2 v[R1];
    float2 u[R2];
    // ---- along z, real to complex: rows 2p and 2p+1 ride as real and imaginary part of line p
    const int np = (ny + 1) >> 1;             // <= N / 2 < ZC lines
    if (in_a) {
        const int ya = 2 * min(la, np - 1);
        const float ma = la < np ? 1.f : 0.f, mb = (la < np && ya + 1 < ny) ? 1.f : 0.f;
        const float* ra = raw + ya * nz;
        const float* rb = raw + min(ya + 1, ny - 1) * nz;
        // rows that fill the transform length: constant offsets, no padding in z
        if (nz == N) {
#pragma unroll
            for (int m = 0; m < R1; ++m) v[m] = make_float2(ra[ja + R2 * m] * ma, rb[ja + R2 * m] * mb);
        } else {
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const int e = ja + R2 * m, ec = min(e, nz - 1);
                const float me = e < nz ? 1.f : 0.f;
                v[m] = make_float2(ra[ec] * (me * ma), rb[ec] * (me * mb));
            }
        }
    }
    __syncthreads();                          // the raw plane has been read: the region becomes the exchange buffer
    if (in_a) TS::step_a(v, la, ja, tws, R);
    __syncthreads();
    if (q < R1) TS::step_b(u, lb, q, R);
    __syncthreads();
    if (q < R1) {
#pragma unroll
        for (int r = 0; r < R2; ++r) R[lb * P + q + R1 * r] = u[r];           // natural order per line
    }
    __syncthreads();
    // ---- along y: one line per oz.  Its sample y = 2l + h is row h of line l above, untangled on the way in:
    // with Z = line l and W = conj(Z[N - oz]), row 0 is (Z[oz] + W) / 2 and row 1 is -i (Z[oz] - W) / 2.  R2 is even,
    // so a thread sees rows of one parity only, and its lines l advance by R2 / 2 per sample: two addresses, then
    // constant offsets.  (Untangling into a plane of its own first cost a pass through LDS each way, a barrier and
    // index arithmetic per element.)
    static_assert(R2 % 2 == 0, "a thread's samples must have one parity");
    if (in_a) {
        const int oz = la;
        const bool odd = ja & 1;
        if (!PACK || oz) {
            const float sg = odd ? -1.f : 1.f;
            const float2* pz = R + (ja >> 1) * P + oz;
            const float2* pw = R + (ja >> 1) * P + (oz ? N - oz : 0);
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const float mk = ja + R2 * m < ny ? 0.5f : 0.f;
                const float2 z = pz[(R2 / 2) * P * m], w = pw[(R2 / 2) * P * m];
                const float pr = fmaf(sg, w.x, z.x) * mk, qi = fmaf(-sg, w.y, z.y) * mk;
                v[m] = odd ? make_float2(qi, -pr) : make_float2(pr, qi);
            }
        } else {
            // line 0 carries oz = 0 (real part) and oz = N / 2 (imaginary part): at these two bins the rows of a
            // line are simply the real and the imaginary part of the line's value
            const float2* pz = R + (ja >> 1) * P;
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const float mk = ja + R2 * m < ny ? 1.f : 0.f;
                const float2 z = pz[(R2 / 2) * P * m], w = pz[(R2 / 2) * P * m + N / 2];
                v[m] = odd ? make_float2(z.y * mk, w.y * mk) : make_float2(z.x * mk, w.x * mk);
            }
        }
    }
    __syncthreads();                          // the lines have been read: the region is the exchange buffer again
    if (in_a) TS::step_a(v, la, ja, tws, R);
    __syncthreads();
    if (q < R1) TS::step_b(u, lb, q, R);
    __syncthreads();
    if (q < R1) {
#pragma unroll
        for (int r = 0; r < R2; ++r) R[lb * P + q + R1 * r] = u[r];
    }
    __syncthreads();
}

template <int R1, int R2>
__global__ __launch_bounds__((fused_nth_fwd<R1, R2>())) __attribute__((amdgpu_waves_per_eu((fused_waves<R1, R2, true>()))))
void k_fwd_zy(FusedFwdArgs a)
{
    using TS = TwoStep<R1, R2>;
    constexpr int N = TS::N, P = TS::P, ZC = N / 2 + 1;
    constexpr bool PACK = fused_fwd_packs(N);
    extern __shared__ float2 lds[];
    float2* tws = lds;                 // [N]
    float2* R = lds + N;               // in turn: raw plane [ny][nz] floats, exchange buffer and lines [NL][P]
    const int t = threadIdx.x, NTH = blockDim.x;
    const int x = blockIdx.x, img = blockIdx.y;
    const Dims& d = a.d;
    const int ny = d.ny, nz = d.nz;
    const float* plane = a.in + (((size_t)img * d.nx + x) * ny) * nz;

    for (int q = t; q < N; q += NTH) tws[q] = a.tw[q];

    // ---- the (y, z) plane, contiguous in the input tensor, into LDS with fully coalesced loads.  (Reading each
    // line's samples straight into the registers of the first step, as the separate z pass does, touches every
    // cache line from four instructions and, for some row lengths, evicts it in between: measured up to 2.8x
    // slower with a whole plane per workgroup.)
    float* raw = reinterpret_cast<float*>(R);
    {
        // a flat copy, rows at their pitch in memory.  (Padding the rows in LDS so that the lines a wave reads
        // together spread over all banks costs index arithmetic per element -- these kernels are bound by issuing
        // instructions, not by LDS -- and was measured 3-8 % slower at almost every length.)
        const int tot = ny * nz;
        for (int i0 = 0; i0 < tot; i0 += 8 * NTH) {
            float r[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) r[k] = plane[min(i0 + k * NTH + t, tot - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + k * NTH + t < tot) raw[i0 + k * NTH + t] = r[k];
        }
    }
    __syncthreads();

    fwd_plane<R1, R2, 1>(tws, R, 0, ny, nz);
    float2* dst = a.dst + (((size_t)img * d.nx + x) * ZC) * N;
    // a wave per row, or per two or four rows where rows are at most 32 or 16 long; rows 0 and N / 2 come out of
    // line 0 = C: (C[oy] + conj(C[N - oy])) / 2 and -i (C[oy] - conj(C[N - oy])) / 2
    constexpr int LW = N <= 16 ? 16 : N <= 32 ? 32 : 64, RPI = 64 / LW;
    for (int l = (t / 64) * RPI + (t % 64) / LW; l < ZC; l += (NTH / 64) * RPI) {
        if (!PACK || (l != 0 && l != N / 2)) {
            for (int e = t % LW; e < N; e += LW) dst[(size_t)l * N + e] = R[l * P + e];
        } else {
            for (int e = t % LW; e < N; e += LW) {
                const float2 c = R[e], m = cconj(R[e ? N - e : 0]);
                dst[(size_t)l * N + e] = l ? cscale(mul_mi(csub(c, m)), 0.5f) : cscale(cadd(c, m), 0.5f);
            }
        }
    }
}

// A value the compiler knows nothing about: what is worked out from it is worked out again, not kept in registers.
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The tables of the lengths below (double precision rounded once, as k_twiddles makes them): working them out took every
// workgroup longer than reading them.
template <int N> struct TwiddleTable { float2 v[N]; };
template <int N> constexpr TwiddleTable<N> make_twiddles()
{
    TwiddleTable<N> t{};
    for (int q = 0; q < N; ++q) {
        // the quadrant, and the place in its first or second half
        const int quadrant = 4 * q / N, r = 4 * q - quadrant * N;
        const bool upper = 2 * r > N;
        const double x = kPi / 2 * (upper ? N - r : r) / N, s0 = ct_sin_series(x), c0 = ct_cos_series(x);
        const double s = upper ? c0 : s0, c = upper ? s0 : c0;           // of the angle in its quadrant
        const double sn = quadrant == 0 ? s : quadrant == 1 ? c : quadrant == 2 ? -s : -c;
        const double cs = quadrant == 0 ? c : quadrant == 1 ? -s : quadrant == 2 ? -c : s;
        t.v[q].x = (float)cs;
        t.v[q].y = (float)-sn;
    }
    return t;
}
template <int N> __device__ const TwiddleTable<N> kTwiddles = make_twiddles<N>();

// exp(-2 pi i q / N), as k_twiddles makes it.
__device__ __forceinline__ float2 twiddle(int q, int N)
{
    double s, c;
    sincospi(2.0 * (double)q / (double)N, &s, &c);
    return make_float2((float)c, (float)(-s));
}

// Small layers of the route below: what launches before the forward kernel would do -- tables, largest kernel magnitudes, the
// kernel transform's z stage, scales -- is done next to it, by workgroups of their own behind the images'.  Launches follow each
// other 3.8 us apart, and none of this depends on another launch once whoever needs the largest magnitudes of the kernels looks
// at the bank itself.  The results are those of the separate kernels (k_twiddles, k_kprep_z, kprep_row_scale), bit for bit.
// cm: the largest finite kernel magnitude of every input image, a wave per image.  Behind a barrier.
__device__ __forceinline__ void bank_max(const float* __restrict__ w, float* cm, int f, int fo, int taps)
{
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6, n = fo * taps;
    for (int i = threadIdx.x >> 6; i < f; i += 2 * nw) {     // two images at a time
        const int i1 = min(i + nw, f - 1);
        float m = 0.f, m1 = 0.f;
        for (int e0 = lane; e0 < n; e0 += 512) {
            float v[8], v1[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const unsigned e = (unsigned)min(e0 + 64 * u, n - 1), j = e / (unsigned)taps;
                const float* p = w + (size_t)(j * (unsigned)f * (unsigned)taps + (e - j * taps));
                v[u] = fabsf(p[i * taps]);
                v1[u] = fabsf(p[i1 * taps]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                m = fmaxf(m, v[u] < INFINITY ? v[u] : 0.f);
                m1 = fmaxf(m1, v1[u] < INFINITY ? v1[u] : 0.f);
            }
        }
#pragma unroll
        for (int o = 32; o; o >>= 1) { m = fmaxf(m, __shfl_xor(m, o)); m1 = fmaxf(m1, __shfl_xor(m1, o)); }
        if (lane == 0) { cm[i] = m; cm[i1] = m1; }
    }
    __syncthreads();
}
__device__ __forceinline__ float all_max(const float* cm, int f)
{
    float m = 0.f;
    for (int i = threadIdx.x & 63; i < f; i += 64) m = fmaxf(m, cm[i]);
#pragma unroll
    for (int o = 32; o; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    return m;
}

// Workgroup r of these: output image r's scale (and, first of them, those of the input images); the tables; the z stage.
template <int N>
__device__ __forceinline__ void prep_small(const FusedFwdArgs& a, int r, float* lds)
{
    const Dims& d = a.d;
    const int t = threadIdx.x, NT = blockDim.x, wave = t >> 6, lane = t & 63, nw = NT >> 6;
    const int taps = d.kx * d.ky * d.kz;
    if (r < a.Mp) {
        float* cm = lds;
        float4* part = reinterpret_cast<float4*>(lds + ((a.f + 3) & ~3));       // [wave] largest, smallest, smallest but zero
        bank_max(a.w, cm, a.f, a.fo, taps);
        const float most = all_max(cm, a.f);
        if (r == 0)
            for (int i = t; i < a.fp; i += NT) {
                const int e = i < a.f ? kprep_col_exp(cm[i], most) : 0;
                a.S.col[i] = __uint_as_float((unsigned)(127 + e) << 23);
                a.S.cinv[i] = __uint_as_float((unsigned)(127 - e) << 23);
            }
        float m = 0.f;
        unsigned lo = ~0u, lo1 = ~0u;
        if (r < a.fo)
            for (int i = wave; i < a.f; i += nw) {
                const float* wi = a.w + ((size_t)r * a.f + i) * taps;
                float s = 0.f;
                for (int t0 = 0; t0 < taps; t0 += 64) s += fabsf(wi[min(t0 + lane, taps - 1)]) * (t0 + lane < taps ? 1.f : 0.f);
#pragma unroll
                for (int o = 32; o; o >>= 1) s += __shfl_xor(s, o);
                const float e = ldexpf(s * a.scale, -kprep_col_exp(cm[i], most));
                m = fmaxf(m, e < INFINITY ? e : 0.f);
                lo = min(lo, __float_as_uint(e));
                lo1 = min(lo1, __float_as_uint(e) - 1u);
            }
        if (lane == 0) part[wave] = make_float4(m, __uint_as_float(lo), __uint_as_float(lo1), 0.f);
        __syncthreads();
        if (t == 0) {
            for (int q = 0; q < nw; ++q) {
                const float4 v = part[q];
                m = fmaxf(m, v.x); lo = min(lo, __float_as_uint(v.y)); lo1 = min(lo1, __float_as_uint(v.z));
            }
            kprep_row_store(a.S, r, m, lo, lo1);
        }
        return;
    }
    if (r == a.Mp) {
        for (int q = t; q < d.Nx; q += NT) a.twx[q] = twiddle(q, d.Nx);
        for (int q = t; q < d.Ny; q += NT) {
            const float2 v = kTwiddles<N>.v[q];              // (Ny = Nz = N here)
            const_cast<float2*>(a.tw)[q] = v;
            a.twz[q] = v;
        }
        return;
    }
    r -= a.Mp + 1;
    const int per = d.ky * d.kx * a.fp * a.Mp, nb = (per + NT - 1) / NT;
    const int oz0 = r / nb * KPREP_OZ, idx = (r - r / nb * nb) * NT + t;
    float2* tw2 = reinterpret_cast<float2*>(lds);            // [taps][KPREP_OZ]
    for (int e = t; e < d.kz * KPREP_OZ; e += NT) {
        const int c = e / KPREP_OZ, o = e - c * KPREP_OZ;
        tw2[e] = kTwiddles<N>.v[(oz0 + o) * c % N];
    }
    __syncthreads();
    if (idx >= per) return;
    const int j = idx % a.Mp, i = (idx / a.Mp) % a.fp, ba = idx / (a.Mp * a.fp), x = ba % d.kx, y = ba / d.kx;
    float2 acc[KPREP_OZ];
#pragma unroll
    for (int o = 0; o < KPREP_OZ; ++o) acc[o] = make_float2(0.f, 0.f);
    if (i < a.f && j < a.fo) {
        const float* wr = a.w + ((((size_t)j * a.f + i) * d.kx + x) * d.ky + y) * d.kz;
        for (int c = 0; c < d.kz; ++c) {
            const float v = wr[c];
#pragma unroll
            for (int o = 0; o < KPREP_OZ; ++o) acc[o] = caxpy(acc[o], v, tw2[c * KPREP_OZ + o]);
        }
    }
#pragma unroll
    for (int o = 0; o < KPREP_OZ; ++o)
        if (oz0 + o < d.zc) a.A1[(size_t)(oz0 + o) * per + idx] = acc[o];
}

// Four neighbouring x at a time (see k_inv_yz_planes): X2 as [img][oz][x / 4][oy][x % 4].
template <int R1, int R2, int PAR_, bool SMALL>
__device__ __forceinline__ void fwd_planes(const FusedFwdArgs& a)
{
    using PL = Planes<R1, R2, PAR_, true>;
    constexpr int N = PL::N, P = N + 2, ZC = N / 2 + 1, NTH = PL::NTH, PAR = PL::PAR, ROUNDS = PL::ROUNDS, RS = PL::RS;
    constexpr int NV = (PAR * ZC * N + NTH - 1) / NTH, NF = (N * N + NTH - 1) / NTH;    // results and raw values of a plane per thread
    extern __shared__ float2 lds[];
    float2* tws = lds;                 // [N]
    float2* R = lds + N;               // per plane, in turn: raw plane [ny][nz] floats, exchange buffer and lines [NL][P]
    const int t = threadIdx.x, xb = blockIdx.x, img = blockIdx.y, nxb = gridDim.x;
    const Dims& d = a.d;
    if (SMALL && img >= a.nimg) {
        prep_small<N>(a, (img - a.nimg) * nxb + xb, reinterpret_cast<float*>(lds));
        return;
    }
    const int tot = d.ny * d.nz, left = d.nx - PLANES * xb;      // planes from this block's first on
    const float* plane = a.in + ((size_t)img * d.nx + PLANES * xb) * tot;
    float ps = 1.f;
    if (!SMALL && a.col) ps = a.col[img % a.f];

    // the planes of a round; the next round's are requested while one is transformed.  (Planes beyond the image repeat its
    // last one, and are never read.)
    float raw[PAR][NF];
    auto request = [&](int h) {
        const int tp = fresh(t);
#pragma unroll
        for (int p = 0; p < PAR; ++p) {
            const float* src = plane + (size_t)min(p * ROUNDS + h, left - 1) * tot;
#pragma unroll
            for (int k = 0; k < NF; ++k) raw[p][k] = src[min(k * NTH + tp, tot - 1)];
        }
    };
    request(0);
    if constexpr (!SMALL) {
        for (int q = t; q < N; q += NTH) tws[q] = a.tw[q];
    } else {
        if (t < N) tws[t] = kTwiddles<N>.v[t];               // (N <= 64 < NTH)
        float* cm = reinterpret_cast<float*>(R + PAR * RS);
        bank_max(a.w, cm, a.f, a.fo, d.kx * d.ky * d.kz);
        ps = __uint_as_float((unsigned)(127 + kprep_col_exp(cm[img % a.f], all_max(cm, a.f))) << 23);
    }
    struct alignas(8 * (ROUNDS > 1 ? 2 : 1)) Run { float2 v[ROUNDS]; } keep[NV];
#pragma unroll
    for (int h = 0; h < ROUNDS; ++h) {
        if (h) __syncthreads();               // the lines have been read: the region takes the next raw plane
        const int tp = fresh(t);
#pragma unroll
        for (int p = 0; p < PAR; ++p)
#pragma unroll
            for (int k = 0; k < NF; ++k)
                if (k * NTH + tp < tot) reinterpret_cast<float*>(R + p * RS)[k * NTH + tp] = raw[p][k];
        __syncthreads();
        if (h + 1 < ROUNDS && h + 1 < left) request(h + 1);
        fwd_plane<R1, R2, PAR>(tws, R, RS, d.ny, d.nz);
        const float2* Rp = R + tp % PAR * RS;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i = min((k * NTH + tp) / PAR, ZC * N - 1), l = i / N, e = i - l * N;
            if (PL::PACK && (l == 0 || l == N / 2)) {
                const float2 c = Rp[e], m = cconj(Rp[e ? N - e : 0]);
                keep[k].v[h] = l ? cscale(mul_mi(csub(c, m)), 0.5f) : cscale(cadd(c, m), 0.5f);
            } else keep[k].v[h] = Rp[l * P + e];
        }
    }
    // neighbouring threads store neighbouring values: whole runs of a row
    float2* dst = a.dst + (((size_t)img * ZC) * nxb + xb) * N * PLANES + t % PAR * ROUNDS;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = (k * NTH + t) / PAR, l = i / N, e = i - l * N;
        if (i >= ZC * N) break;
#pragma unroll
        for (int h = 0; h < ROUNDS; ++h) { keep[k].v[h].x *= ps; keep[k].v[h].y *= ps; }
        *reinterpret_cast<Run*>(dst + ((size_t)l * nxb * N + e) * PLANES) = keep[k];
    }
}

template <int R1, int R2, int PAR>
__global__ __launch_bounds__((Planes<R1, R2, PAR, true>::NTH)) __attribute__((amdgpu_waves_per_eu((Planes<R1, R2, PAR, true>::WAVES))))
void k_fwd_zy_planes(FusedFwdArgs a)
{
    fwd_planes<R1, R2, PAR, false>(a);
}
// ... with the kernels' first stage beside it (all four planes at once: few workgroups)
template <int R1, int R2>
__global__ __launch_bounds__((Planes<R1, R2, PLANES, true>::NTH)) void k_fwd_zy_small(FusedFwdArgs a)
{
    fwd_planes<R1, R2, PLANES, true>(a);
}

// ------------------------------------------------------------------------------------------- host side
struct FusedShape { int R1, R2, QP, RP, nth; size_t lds; };

// The in-register split of each supported length, measured best per length (32 -> 32 images, batches of 1.5 GB):
// mostly R1 x 8 -- fewer, fatter threads than the separate passes use would not cover a plane's lines in one
// round --, with the squarer splits 6 x 6, 8 x 10 and 8 x 12 10 to 15 % ahead at 36, 80 and 96.  At 120 both
// kernels take 10 x 12 (12 threads per line instead of 15): the inverse kernel then runs two workgroups per CU instead
// of one and is 40 % faster, the forward kernel is 10 % faster with it than with 15 x 8.
static bool fused_split(int N, bool forward, int* R1, int* R2)
{
    static const int tab[][3] = {{8, 2, 4},    {10, 5, 2},  {12, 3, 4},  {14, 7, 2},  {16, 4, 4},  {20, 5, 4},
                                 {24, 6, 4},   {28, 7, 4},  {32, 4, 8},  {36, 6, 6},  {40, 5, 8},  {48, 6, 8},
                                 {56, 7, 8},   {64, 8, 8},  {72, 9, 8},  {80, 8, 10}, {96, 8, 12}, {100, 10, 10},
                                 {112, 7, 16}, {120, 15, 8}};
    if (N == 120) { *R1 = 10; *R2 = 12; return true; }
    if (N == 128 && forward) { *R1 = 8; *R2 = 16; return true; }    // one round of 1024 threads: 64 lines x 16
    for (const auto& e : tab)
        if (e[0] == N) { *R1 = e[1]; *R2 = e[2]; return true; }
    return false;
}

// forward = true: the plane holds ny columns instead of noy, and the x pass after it must be an in-register one
static bool fused_shape(const LayerPlan& L, FusedShape* F, bool forward = false)
{
    const Dims& d = L.d;
    if (L.generic_passes || d.Ny != d.Nz) return false;
    int R1, R2;
    if (!fused_split(d.Ny, forward, &R1, &R2)) return false;
    F->R1 = R1; F->R2 = R2;
    if (forward) {
        if (!fast_pass_available(d.Nx) || d.nx > 65535 || L.nimg > 65535) return false;
    } else {
        if (d.nox > 65535 || L.nimgo > 65535) return false;
    }
    const int N = d.Ny, zc = d.zc;
    const int cols = forward ? d.ny : d.noy;
    F->QP = cols + 2 - (cols & 1);
    F->RP = d.nz;
    const int lines = (forward ? fused_fwd_packs(N) : fused_inv_packs(N)) ? N / 2 : zc;   // two lines may ride as one
    F->nth = (lines * std::max(R1, R2) + 63) / 64 * 64;
    size_t region = sizeof(float2) * (size_t)(forward ? lines : zc) * (N + 2);      // the inverse plane Q has zc rows
    if (forward) region = std::max(region, sizeof(float) * (size_t)d.ny * F->RP);
    F->lds = sizeof(float2) * (size_t)N + region;
    return F->nth <= 1024 && F->lds <= 80 * 1024;             // two workgroups per CU at least
}

bool fused_inv_yz_available(const LayerPlan& L)
{
    FusedShape F;
    return fused_shape(L, &F);
}

bool fused_fwd_zy_available(const LayerPlan& L)
{
    FusedShape F;
    return fused_shape(L, &F, true);
}

template <typename Args>
static znni_status launch_fused(void (*kernel)(Args), const Args& a, const FusedShape& F, dim3 grid, hipStream_t st)
{
    if (F.lds > 48 * 1024 &&
        hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)F.lds) != hipSuccess)
        return ZNNI_ERR_HIP;
    kernel<<<grid, dim3(F.nth), F.lds, st>>>(a);
    if (hipGetLastError() != hipSuccess) return ZNNI_ERR_HIP;
    return ZNNI_OK;
}

// dispatch on the split that fused_split chose (R1 * 100 + R2)
#define ZNNI_FUSED_CASES(KERNEL)                                                                   \
    switch (F.R1 * 100 + F.R2) {                                                                   \
        case 204: return launch_fused(KERNEL<2, 4>, a, F, grid, st);                               \
        case 502: return launch_fused(KERNEL<5, 2>, a, F, grid, st);                               \
        case 304: return launch_fused(KERNEL<3, 4>, a, F, grid, st);                               \
        case 702: return launch_fused(KERNEL<7, 2>, a, F, grid, st);                               \
        case 404: return launch_fused(KERNEL<4, 4>, a, F, grid, st);                               \
        case 504: return launch_fused(KERNEL<5, 4>, a, F, grid, st);                               \
        case 604: return launch_fused(KERNEL<6, 4>, a, F, grid, st);                               \
        case 704: return launch_fused(KERNEL<7, 4>, a, F, grid, st);                               \
        case 408: return launch_fused(KERNEL<4, 8>, a, F, grid, st);                               \
        case 606: return launch_fused(KERNEL<6, 6>, a, F, grid, st);                               \
        case 508: return launch_fused(KERNEL<5, 8>, a, F, grid, st);                               \
        case 608: return launch_fused(KERNEL<6, 8>, a, F, grid, st);                               \
        case 708: return launch_fused(KERNEL<7, 8>, a, F, grid, st);                               \
        case 808: return launch_fused(KERNEL<8, 8>, a, F, grid, st);                               \
        case 908: return launch_fused(KERNEL<9, 8>, a, F, grid, st);                               \
        case 810: return launch_fused(KERNEL<8, 10>, a, F, grid, st);                              \
        case 812: return launch_fused(KERNEL<8, 12>, a, F, grid, st);                              \
        case 1010: return launch_fused(KERNEL<10, 10>, a, F, grid, st);                            \
        case 716: return launch_fused(KERNEL<7, 16>, a, F, grid, st);                              \
        case 1508: return launch_fused(KERNEL<15, 8>, a, F, grid, st);                             \
        case 1012: return launch_fused(KERNEL<10, 12>, a, F, grid, st);                            \
        case 816: return launch_fused(KERNEL<8, 16>, a, F, grid, st);                              \
    }                                                                                              \
    return ZNNI_ERR_UNSUPPORTED_SIZE;

// in -> X2' (buf1); to be followed by launch_fast_fwd_xt
znni_status launch_fwd_zy(const LayerPlan& L, const float* in, hipStream_t st)
{
    FusedShape F;
    if (!fused_shape(L, &F, true)) return ZNNI_ERR_UNSUPPORTED_SIZE;
    const Dims& d = L.d;
    FusedFwdArgs a;
    a.in = in; a.dst = L.buf1; a.tw = L.twy; a.d = d;
    a.col = nullptr; a.f = 1; a.w = nullptr;
    const dim3 grid(d.nx, L.nimg);
    ZNNI_FUSED_CASES(k_fwd_zy)
}

znni_status launch_inv_yz(const LayerPlan& L, const float* bias, float* out, unsigned flags, hipStream_t st)
{
    FusedShape F;
    if (!fused_shape(L, &F)) return ZNNI_ERR_UNSUPPORTED_SIZE;
    const Dims& d = L.d;
    FusedArgs a;
    a.src = L.buf0; a.out = out; a.tw = L.twy; a.bias = bias;
    a.d = d; a.fo = L.fo; a.relu = (flags & ZNNI_RELU) ? 1 : 0;
    a.QP = F.QP;
    const dim3 grid(d.nox, L.nimgo);
    ZNNI_FUSED_CASES(k_inv_yz)
}

// The kernels for four planes: threads and LDS of a workgroup.
static bool planes_shape(const LayerPlan& L, FusedShape* F, bool forward, int* together = nullptr)
{
    if (!fused_shape(L, F, forward)) return false;
    const int N = L.d.Ny;
    const bool packs = forward ? fused_fwd_packs(N) : fused_inv_packs(N);
    const long long groups = ((forward ? L.d.nx : L.d.nox) + PLANES - 1) / PLANES * (long long)(forward ? L.nimg : L.nimgo);
    const int lines = packs ? N / 2 : L.d.zc, par = planes_wide(N, packs) || groups < PLANES_FEW ? PLANES : 1;
    if (together) *together = par;
    F->nth = planes_nth(lines, std::max(F->R1, F->R2), par);
    F->lds = sizeof(float2) * (size_t)(N + par * planes_pitch((forward ? lines : L.d.zc) * (N + 2)));
    return N <= PLANES_MAX && F->nth <= 1024 && F->lds <= 80 * 1024;
}

bool fused_planes_available(const LayerPlan& L)
{
    FusedShape F;
    return planes_shape(L, &F, true) && planes_shape(L, &F, false);
}

template <int R1, int R2>
static znni_status launch_planes(const FusedFwdArgs& a, const FusedShape& F, int par, dim3 grid, hipStream_t st)
{
    if (a.w) return launch_fused(k_fwd_zy_small<R1, R2>, a, F, grid, st);
    if constexpr (!planes_wide(R1 * R2, fused_fwd_packs(R1 * R2)))
        if (par == 1) return launch_fused(k_fwd_zy_planes<R1, R2, 1>, a, F, grid, st);
    return launch_fused(k_fwd_zy_planes<R1, R2, PLANES>, a, F, grid, st);
}
template <int R1, int R2>
static znni_status launch_planes(const FusedArgs& a, const FusedShape& F, int par, dim3 grid, hipStream_t st)
{
    if constexpr (!planes_wide(R1 * R2, fused_inv_packs(R1 * R2)))
        if (par == 1) return launch_fused(k_inv_yz_planes<R1, R2, 1>, a, F, grid, st);
    return launch_fused(k_inv_yz_planes<R1, R2, PLANES>, a, F, grid, st);
}
template <typename Args>
static znni_status launch_planes(const Args& a, const FusedShape& F, int par, dim3 grid, hipStream_t st)
{
    switch (F.R1 * 100 + F.R2) {
        case 204: return launch_planes<2, 4>(a, F, par, grid, st);
        case 502: return launch_planes<5, 2>(a, F, par, grid, st);
        case 304: return launch_planes<3, 4>(a, F, par, grid, st);
        case 702: return launch_planes<7, 2>(a, F, par, grid, st);
        case 404: return launch_planes<4, 4>(a, F, par, grid, st);
        case 504: return launch_planes<5, 4>(a, F, par, grid, st);
        case 604: return launch_planes<6, 4>(a, F, par, grid, st);
        case 704: return launch_planes<7, 4>(a, F, par, grid, st);
        case 408: return launch_planes<4, 8>(a, F, par, grid, st);
        case 606: return launch_planes<6, 6>(a, F, par, grid, st);
        case 508: return launch_planes<5, 8>(a, F, par, grid, st);
        case 608: return launch_planes<6, 8>(a, F, par, grid, st);
        case 708: return launch_planes<7, 8>(a, F, par, grid, st);
        case 808: return launch_planes<8, 8>(a, F, par, grid, st);
    }
    return ZNNI_ERR_UNSUPPORTED_SIZE;
}

static size_t prep_small_lds(const LayerPlan& L, int nth)
{
    const size_t scale = sizeof(float) * ((L.f + 3) & ~3) + sizeof(float4) * (nth / 64), z = sizeof(float2) * L.d.kz * KPREP_OZ;
    return std::max(scale, z);
}
// Whether a layer is small enough for every workgroup of the forward kernel to look at the kernel bank by itself: turns of a wave
// over the bank, eight values a lane at a time, against the two launches that it saves.  Over 2200 random layers of up to 7
// inputs and fewer than PLANES_FEW workgroups, against launches of their own: one turn 1.18 times as fast, 2 or 3 1.16, 4 to 8 1.09, 9 to 16
// 0.99, more 0.6 to 0.85; with more waves than the chip has SIMDs, all of which look at the bank, each a little less (three times as
// many: 1.05, 1.04, 0.98).  Batches are left out: their transforms fill the chip.
bool prep_small_available(const LayerPlan& L)
{
    FusedShape F;
    int par = 0;
    if (!L.planes || L.tiles || L.S >= 8 || !planes_shape(L, &F, true, &par) || par != PLANES) return false;
    const int nw = F.nth / 64;
    const long long turns = (long long)((L.f + nw - 1) / nw) * ((L.fo * L.d.kx * L.d.ky * L.d.kz + 511) / 512);
    const long long waves = (long long)L.nimg * ((L.d.nx + PLANES - 1) / PLANES) * nw;
    return turns * std::max(waves, 1024ll) <= 8 * 1024;
}

// in -> X2 in blocks of four x (buf1); Yd in blocks of four xo (Yt) -> out.  w: with the kernels' z stage, scales and tables.
znni_status launch_fwd_zy_planes(const LayerPlan& L, const float* in, const float* w, hipStream_t st)
{
    if (L.tiles) return launch_fwd_tiles(L, in, st);
    FusedShape F;
    int par = 1;
    if (!planes_shape(L, &F, true, &par)) return ZNNI_ERR_UNSUPPORTED_SIZE;
    const Dims& d = L.d;
    FusedFwdArgs a;
    a.in = in; a.dst = L.buf1; a.tw = L.twy; a.d = d;
    a.col = split_scales(L).col; a.f = L.f;
    a.w = w; a.A1 = L.A1; a.twx = L.twx; a.twz = L.twz; a.S = split_scales(L);
    a.nimg = L.nimg; a.fo = L.fo; a.fp = L.fp; a.Mp = L.Mp; a.scale = (float)(1.0 / ((double)d.Ny * d.Nz));
    dim3 grid((d.nx + PLANES - 1) / PLANES, L.nimg);
    if (w) {
        F.lds = std::max(F.lds + sizeof(float) * L.f, prep_small_lds(L, F.nth));
        const int per = d.ky * d.kx * L.fp * L.Mp;
        const long long more = L.Mp + 1 + (long long)((per + F.nth - 1) / F.nth) * ((d.zc + KPREP_OZ - 1) / KPREP_OZ);
        if (F.lds > 160 * 1024 || L.nimg + (more + grid.x - 1) / grid.x > 65535) return ZNNI_ERR_SHAPE;
        grid.y += (unsigned)((more + grid.x - 1) / grid.x);
    }
    return launch_planes(a, F, par, grid, st);
}

znni_status launch_inv_yz_planes(const LayerPlan& L, const float* bias, float* out, unsigned flags, hipStream_t st)
{
    if (L.tiles) return launch_inv_tiles(L, bias, out, flags, st);
    FusedShape F;
    int par = 1;
    if (!planes_shape(L, &F, false, &par)) return ZNNI_ERR_UNSUPPORTED_SIZE;
    const Dims& d = L.d;
    FusedArgs a;
    a.src = L.Yt; a.out = out; a.tw = L.twy; a.bias = bias;
    a.d = d; a.fo = L.fo; a.relu = (flags & ZNNI_RELU) ? 1 : 0;
    a.QP = F.QP;
    const dim3 grid((d.nox + PLANES - 1) / PLANES, L.nimgo);
    return launch_planes(a, F, par, grid, st);
}

}  // namespace znni
