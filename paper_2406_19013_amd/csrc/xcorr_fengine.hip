// F-engine front end (paper Section 2.2): 8-bit ADC samples of each input ->
// polyphase filter bank of 2048 points with a 4-tap prototype -> real FFT ->
// 1024 channels -> per-(input, channel) EQ gain -> 4+4-bit requantisation ->
// corner turn into the X-engine's [T][F][N] order.
//
// Persistent work-groups of 8 waves (two per SIMD); an item is one spectrum,
// or two consecutive ones, of 16 inputs, 2 per wave.  A wave filters and
// transforms an input's one or two spectra in lockstep.  Per input and
// spectrum:
//   y[q] = sum_k h[k P + q] x[(m + k) P + q]            q < P = 2048
//   z[n] = y[2n] + i y[2n + 1]                          n < 1024
//   Z    = 1024-point complex DFT of z (radix 16 x 16 x 4)
//   Y[c] = (Z[c] + Z*[N - c]) / 2 - i W^c (Z[c] - Z*[N - c]) / 2,  W = e^{-2 pi i / 2048}
//   code = pack(clip(rint(g Re Y)), clip(rint(g Im Y)))  for channels c < 1024
// A lane reads 32 consecutive samples of each tap with 16-byte loads (one
// input ahead of the one it transforms); the prototype is copied into LDS
// once per work-group, ordered so that the 128 coefficients of a lane's sample
// positions come as 32 conflict-free 16-byte reads (held in registers they
// took 512 per lane and left room for one wave per SIMD); three full LDS
// exchanges per transform (into the stride-64 order and between the three
// radix passes) and half of one for the Z[N - c] pairs.  Twiddles are built
// per lane from one base value by short power products (at most three
// roundings deep).  The 16 inputs' codes are gathered in LDS and leave as one
// 16-byte row per (spectrum, channel).  Arithmetic in fp32; rounding is
// round-half-to-even.
//
// What bounds it: vector arithmetic (79 % of the cycles issue it), then the
// LDS exchanges.  Two spectra at once share the coefficient reads, three of
// every four sample conversions' blocks, the twiddle powers and the gains:
// 1,136 vector instructions per transform instead of 1,600.  192 inputs x
// 4096 spectra: 2.84 ms with one spectrum at a time; 2.37 ms with two, no
// waits inside an exchange (a wave's LDS accesses execute in order) and pairs
// Y[c], Y[N - c] formed together; 2.10 ms with exchange layouts free of bank
// conflicts; 1.94 ms with 16-byte exchange reads (LDS busy 57 -> 43 % of the
// cycles).  The rounding of every step is as in the one-spectrum kernel, so the
// codes are the same bytes.
#include "xcorr.h"
#include "xcorr_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

namespace xc {
namespace {

constexpr int kFeP = 2048;          // real points per spectrum
constexpr int kFeN = kFeP / 2;      // complex FFT size and channel count
constexpr int kFeTaps = 4;
constexpr int kFeGroup = 16;        // inputs per item
constexpr int kFeWaves = 8;
constexpr int kFeThreads = 64 * kFeWaves;
constexpr int kFeInputsPerWave = kFeGroup / kFeWaves;
constexpr int kFeWgsPerCu = 1;   // 8 waves: two per SIMD, up to 256 registers each
constexpr int kFeBufFloats = 2 * 1088;              // per wave: the widest exchange (32 rows of 34 float2)
constexpr int kFeCodeStride = 20;                   // bytes per channel row of the code tile (16 + pad)
constexpr int kFeSmemProto = kFeTaps * kFeP * 4;    // the prototype, 32 KB

// ---- twiddle tables, computed at compile time in double ----------------------

// sin and cos of 2 pi num / den: quarter turns split off exactly in integer
// arithmetic, the remaining angle (below pi / 2) by Taylor series (16 terms
// reach double precision there)
struct SinCos {
    double s, c;
};
constexpr SinCos sincos_series(double t)
{
    double s = 0, c = 0, term_s = t, term_c = 1;
    for (int k = 0; k < 16; ++k) {
        s += term_s;
        c += term_c;
        term_s *= -t * t / ((2 * k + 2) * (2 * k + 3));
        term_c *= -t * t / ((2 * k + 1) * (2 * k + 2));
    }
    return {s, c};
}
constexpr SinCos sincos_turn(long num, long den)
{
    constexpr double kTwoPi = 6.283185307179586476925286766559;
    num %= den;
    if (num < 0)
        num += den;
    const long q = (4 * num) / den;           // quarter turns
    const long r = 4 * num - q * den;         // remainder, in units of 1 / (4 den) turn
    const SinCos b = sincos_series(kTwoPi * (double)r / (4.0 * den));
    switch (q) {
    case 0: return {b.s, b.c};
    case 1: return {b.c, -b.s};
    case 2: return {-b.s, -b.c};
    default: return {-b.c, b.s};
    }
}

template <int COUNT>
struct Table {
    float re[COUNT];
    float im[COUNT];
};
// W_den^e = exp(-2 pi i e / den) for e < COUNT
template <int COUNT>
constexpr Table<COUNT> make_powers(long den)
{
    Table<COUNT> t{};
    for (int e = 0; e < COUNT; ++e) {
        const SinCos v = sincos_turn(e, den);
        t.re[e] = (float)v.c;
        t.im[e] = (float)-v.s;
    }
    return t;
}
__device__ constexpr Table<64> kW1024 = make_powers<64>(1024);   // pass-1 bases W1024^l
__device__ constexpr Table<4> kW64 = make_powers<4>(64);         // pass-2 bases W64^m2
__device__ constexpr Table<64> kW2048 = make_powers<64>(2048);   // real-unpack bases W2048^l
constexpr Table<16> kW32 = make_powers<16>(32);                  // W2048^(64 v) = W32^v

// ---- complex helpers ----------------------------------------------------------
//
// The rounding of every product is written out (which of the two products of
// a complex multiplication is fused): a code may sit on a rounding boundary of
// the requantiser, and the same bytes must come out whatever the compiler
// would contract, in the one- and the two-spectrum kernel alike.
#pragma clang fp contract(off)

struct cf {
    float r, i;
};
__device__ __forceinline__ cf cadd(cf a, cf b) { return {a.r + b.r, a.i + b.i}; }
__device__ __forceinline__ cf csub(cf a, cf b) { return {a.r - b.r, a.i - b.i}; }
__device__ __forceinline__ cf cmul_mi(cf a) { return {a.i, -a.r}; }   // a * (-i)
// a b, the imaginary part fused on a.r b.i (cmul_f) or on a.i b.r (cmul_g)
__device__ __forceinline__ cf cmul_f(cf a, cf b)
{
    return {fmaf(a.r, b.r, -(a.i * b.i)), fmaf(a.r, b.i, a.i * b.r)};
}
__device__ __forceinline__ cf cmul_g(cf a, cf b)
{
    return {fmaf(a.r, b.r, -(a.i * b.i)), fmaf(a.i, b.r, a.r * b.i)};
}

// p[k] = w^k for k < 16: w, w^2, w^3 and w^4, w^8, w^12, then products
// (each power at most three roundings from w)
__device__ __forceinline__ void powers16(cf w, cf (&p)[16])
{
    auto square = [](cf a) { return cf{fmaf(a.r, a.r, -(a.i * a.i)), a.r * a.i + a.r * a.i}; };
    p[0] = cf{1.f, 0.f};
    p[1] = w;
    p[2] = square(w);
    p[3] = cmul_f(p[2], w);
    p[4] = square(p[2]);
    p[8] = square(p[4]);
    p[12] = cmul_f(p[8], p[4]);
#pragma unroll
    for (int a = 4; a < 16; a += 4)
#pragma unroll
        for (int b = 1; b < 4; ++b)
            p[a + b] = cmul_g(p[a], p[b]);
}
// z times its twiddle w^k
__device__ __forceinline__ cf twiddle(cf z, const cf (&p)[16], int k)
{
    if (k == 0)
        return {fmaf(z.i, -0.f, z.r), fmaf(z.r, 0.f, z.i)};
    return k == 8 ? cmul_f(z, p[k]) : cmul_g(z, p[k]);
}

// forward 4-point DFT in place: x[k] = sum_n x[n] (-i)^{nk}
__device__ __forceinline__ void dft4(cf &x0, cf &x1, cf &x2, cf &x3)
{
    const cf a = cadd(x0, x2), b = csub(x0, x2), c = cadd(x1, x3), d = cmul_mi(csub(x1, x3));
    x0 = cadd(a, c);
    x2 = csub(a, c);
    x1 = cadd(b, d);
    x3 = csub(b, d);
}

// forward 16-point DFT of x[0..15] in place (4 x 4 with W16 twiddles); the
// output is in natural order
__device__ __forceinline__ void dft16(cf *x)
{
    // n = 4a + b: 4-point DFTs over a for each b -> U[b][c] at x[4c + b]
#pragma unroll
    for (int b = 0; b < 4; ++b)
        dft4(x[b], x[4 + b], x[8 + b], x[12 + b]);
    // twiddles W16^{b c} = exp(-2 pi i b c / 16); x * (re, im) with the fused
    // product the one of x.i (mul_i) or of x.r (mul_r)
    constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508978f, r2 = 0.70710678118654752f;
    auto mul_i = [](cf a, float re, float im) { return cf{fmaf(a.i, -im, re * a.r), fmaf(a.i, re, im * a.r)}; };
    auto mul_r = [](cf a, float re, float im) { return cf{fmaf(a.r, re, -(im * a.i)), fmaf(a.r, im, re * a.i)}; };
    x[5] = mul_i(x[5], c1, -s1);
    x[9] = mul_i(x[9], r2, -r2);
    x[13] = mul_i(x[13], s1, -c1);
    x[6] = mul_i(x[6], r2, -r2);
    x[10] = cmul_mi(x[10]);
    x[14] = mul_i(x[14], -r2, -r2);
    x[7] = mul_i(x[7], s1, -c1);
    x[11] = mul_r(x[11], -r2, -r2);
    x[15] = mul_r(x[15], -c1, s1);
    // 4-point DFTs over b for each c: X[c + 4 d] from x[4c + b]
    cf y[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        cf a0 = x[4 * c], a1 = x[4 * c + 1], a2 = x[4 * c + 2], a3 = x[4 * c + 3];
        dft4(a0, a1, a2, a3);
        y[c] = a0;
        y[c + 4] = a1;
        y[c + 8] = a2;
        y[c + 12] = a3;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
        x[k] = y[k];
}

// W2048^(lane + 64 v) = W2048^lane W32^v, with the roundings of the
// per-lane products the unpack step was first written with
__device__ __forceinline__ cf unpack_twiddle(cf wl, int v)
{
    if (v == 0)
        return wl;
    const cf k{kW32.re[v], kW32.im[v]};
    const bool alt = v >= 9 && v <= 11;
    const float r = alt ? fmaf(wl.i, -k.i, k.r * wl.r) : fmaf(wl.r, k.r, -(wl.i * k.i));
    const float i = v >= 9 && v <= 12 ? fmaf(wl.r, k.i, wl.i * k.r) : fmaf(wl.i, k.r, wl.r * k.i);
    return {r, i};
}

// A wave's LDS accesses are executed in order, so an exchange between its
// lanes needs no wait between the writes and the reads (nor before the next
// exchange overwrites the buffer): the fence only keeps the compiler from
// moving accesses across it.
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// work-group barrier that waits for this wave's LDS accesses only (the loads
// of the next samples and the stores of the codes stay in flight)
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The packed code of one channel: re and im scaled, clipped to [-8, 7] and
// rounded half to even (clipping first gives the same: the bounds are whole).
// Adding 1.5 2^23 rounds to a whole number whose low bits are the sum's.
__device__ __forceinline__ uint32_t pack_code(float g, cf y)
{
    constexpr float kRound = 12582912.0f;
    const float re = fminf(fmaxf(g * y.r, -8.0f), 7.0f) + kRound;
    const float im = fminf(fmaxf(g * y.i, -8.0f), 7.0f) + kRound;
    return (__builtin_bit_cast(uint32_t, re) << 4) | (__builtin_bit_cast(uint32_t, im) & 15u);
}

struct FeArgs {
    const int8_t *adc;    // [N][S]
    int64_t S;            // samples per input
    int N;
    const float *h;       // [taps * P]
    const float *gains;   // [N][1024]
    int n_spectra;
    void *out;            // CODES: uint8 [n_spectra][1024][N]; else float2 [N][n_spectra][1024]
};

// Raw samples for NS consecutive spectra from m: this lane's 32 consecutive
// samples of the blocks m .. m + NS + 2 (2048 samples each) as two 16-byte
// loads a block; blocks past the last spectrum's are that spectrum's again.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <int NS>
struct FeRaw {
    u32x4 v[kFeTaps + NS - 1][2];
};
template <int NS>
__device__ __forceinline__ void fe_load(const FeArgs &a, int input, int m, FeRaw<NS> &r)
{
    const int lane = threadIdx.x & 63;
    const u32x4 *x = (const u32x4 *)(a.adc + (int64_t)input * a.S + (int64_t)m * kFeP + 32 * lane);
    const int last = a.n_spectra - 1 - m + kFeTaps - 1;   // last block a spectrum needs
#pragma unroll
    for (int k = 0; k < kFeTaps + NS - 1; ++k) {
        const int b = k < kFeTaps ? k : min(k, last);
        r.v[k][0] = x[b * (kFeP / 16)];
        r.v[k][1] = x[b * (kFeP / 16) + 1];
    }
}

__device__ __forceinline__ float byte_at(const u32x4 &v, int t)
{
    const uint32_t w = t < 4 ? v.x : t < 8 ? v.y : t < 12 ? v.z : v.w;
    return (float)(int8_t)(w >> (8 * (t & 3)));
}

// FIR of this lane's 32 samples of NS consecutive spectra -> z[s][j] for
// n = 16 lane + j; samples 4 t4 .. 4 t4 + 3 make z[2 t4] and z[2 t4 + 1].
// hl: the prototype in LDS, float4 (k, t4, lane) = h[k P + 32 lane + 4 t4 ..];
// each coefficient read and each converted sample serves every spectrum that
// uses it.
template <int NS>
__device__ __forceinline__ void fe_fir(const FeRaw<NS> &raw, const float4 *hl, cf (&z)[NS][16])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t4 = 0; t4 < 8; ++t4) {
        // The coefficient reads are the same for every transform: left alone
        // the compiler hoists or clusters all 32 (128 registers live at
        // once).  An opaque offset behind a memory clobber keeps each group
        // of four between its neighbours.
        int l = lane;
        asm volatile("" : "+v"(l) : : "memory");
        float4 h[kFeTaps];
#pragma unroll
        for (int k = 0; k < kFeTaps; ++k)
            h[k] = hl[(k * 8 + t4) * 64 + l];
        float4 y[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s)
            y[s] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int b = 0; b < kFeTaps + NS - 1; ++b) {
            const u32x4 &v = raw.v[b][t4 >> 2];
            const int t = (4 * t4) & 15;
            const float x0 = byte_at(v, t), x1 = byte_at(v, t + 1), x2 = byte_at(v, t + 2), x3 = byte_at(v, t + 3);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int k = b - s;
                if (k >= 0 && k < kFeTaps) {
                    y[s].x = fmaf(h[k].x, x0, y[s].x);
                    y[s].y = fmaf(h[k].y, x1, y[s].y);
                    y[s].z = fmaf(h[k].z, x2, y[s].z);
                    y[s].w = fmaf(h[k].w, x3, y[s].w);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            z[s][2 * t4] = cf{y[s].x, y[s].y};
            z[s][2 * t4 + 1] = cf{y[s].z, y[s].w};
        }
    }
}

struct FeBases {
    cf w1024, w64;   // W1024^lane, W64^(lane / 16)
};

// The FFT of NS spectra of one input by one wave, in lockstep (the twiddles
// are formed once, and one spectrum's exchange runs under the other's
// arithmetic); halfway() is called between the passes, then emit(s, v, second, y) for the channels c = lane + 64 v,
// v < 8 (second = false), and their partners 1024 - c (second = true); lane
// 0's partner for v = 0 is channel 512.
// buf: this wave's exchange buffer; wt: the unpack twiddles (see kFeWtEntries).
// The layouts give 16-byte reads (measured 5.7 cycles for 64 lanes, against 8
// to 16 for the ds_read2_b64 that pairs of 8-byte reads become) and writes
// whose 16 lanes at a time fall on distinct bank pairs.
template <int NS, class Halfway, class Emit>
__device__ __forceinline__ void fe_fft(cf (&z)[NS][16], const FeBases &bs, float2 *buf, const float2 *wt,
                                       Halfway &&halfway, Emit &&emit)
{
    // the exchange addresses are the same for every transform; an opaque lane
    // makes the compiler form them here instead of keeping them live across
    // the loop
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    // likewise the twiddles derived from the per-lane bases
    FeBases b = bs;
    asm volatile("" : "+v"(b.w1024.r), "+v"(b.w1024.i), "+v"(b.w64.r), "+v"(b.w64.i));
    const int k1 = lane & 15, m2 = lane >> 4;   // passes 2 and 3 (m2 is r there)
    // Exchanges 0 and 1 move a 64 x 16 matrix M[16 g + j][a] whose row
    // a = 4.. has its g, j spread over lanes: written by lane 4 a + g (element
    // j at 2 (16 g + j) + a % 2, padded), read by lane 16 g + j, two values of
    // a to a 16-byte read.
    float2 *const w0 = buf + 34 * (lane & 3) + ((lane >> 2) & 1) + 136 * (lane >> 3);
    const float4 *const r0 = (const float4 *)(buf + 2 * lane + 2 * (lane >> 4));
    // exchange 0: lane l holds z[16 l + j]; lane l takes z[64 n1 + l]
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int j = 0; j < 16; ++j)
            w0[2 * j] = make_float2(z[s][j].r, z[s][j].i);
        wave_order();
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const float4 v = r0[68 * n];
            z[s][2 * n] = cf{v.x, v.y};
            z[s][2 * n + 1] = cf{v.z, v.w};
        }
        wave_order();
    }
    // pass 1: 16-point DFT over n1 (n = 64 n1 + l), twiddle W1024^{l k1};
    // lane l holds A[l][k1]
    // pass 2: lane = (m2, k1); 16-point DFT over m1 of A[4 m1 + m2][k1], twiddle W64^{m2 j1};
    // B[k1][m2][j1] at 2 (16 (j1 % 4) + k1) + m2 % 2, rows (m2 / 2, j1 / 4)
    float2 *const w2 = buf + 2 * k1 + (m2 & 1) + 512 * (m2 >> 1);
    const float4 *const r2 = (const float4 *)(buf + 2 * lane);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        cf tw[16];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            dft16(z[s]);
            if (s == 0)
                powers16(pass ? b.w64 : b.w1024, tw);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const cf v = twiddle(z[s][k], tw, k);
                (pass ? w2[32 * (k & 3) + 128 * (k >> 2)] : w0[2 * k]) = make_float2(v.r, v.i);
            }
            wave_order();
            // pass 3 takes j1 = r + 4 u, q = m2 of its k1, at 4 u + q
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const float4 v = pass ? r2[64 * (n >> 1) + 256 * (n & 1)] : r0[68 * n];
                z[s][2 * n] = cf{v.x, v.y};
                z[s][2 * n + 1] = cf{v.z, v.w};
            }
            wave_order();
        }
        if (pass == 0)
            halfway();
    }
    // pass 3: lane = (r, k1); for j1 = r + 4 u: 4-point DFT over q -> Z[k1 + 16 j1 + 256 j2],
    // that is Z[lane + 64 v], v = u + 4 j2: every lane already holds its
    // channels c = lane + 64 v; the partners 1024 - c = (64 - lane) + 64 (15 - v)
    // of v < 8 come from lane 64 - lane
    float2 *const lin = buf + lane;
    const float2 *const rev = buf + 64 - lane;
    const float4 *const wlin = (const float4 *)(wt + 2 * lane), *const wrev = (const float4 *)(wt + 128 - 2 * lane);
    cf zn[NS][8];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            cf *q = &z[s][4 * u];   // Z[lane + 64 (u + 4 j2)] at 4 u + j2
            dft4(q[0], q[1], q[2], q[3]);
            lin[64 * u] = make_float2(q[2].r, q[2].i);
            lin[64 * u + 256] = make_float2(q[3].r, q[3].i);
        }
        wave_order();
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            // (lane 0, v = 0 has no partner row: see below)
            const float2 q = rev[v == 0 && lane == 0 ? 0 : 64 * (7 - v)];
            zn[s][v] = cf{q.x, q.y};
        }
        wave_order();
    }
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        const float4 w4 = wlin[65 * (v >> 1)], x4 = wrev[65 * (7 - (v >> 1))];
        const cf wa = v & 1 ? cf{w4.z, w4.w} : cf{w4.x, w4.y};
        const cf wb = v & 1 ? cf{x4.x, x4.y} : cf{x4.z, x4.w};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // Y[c] = (Z[c] + Z*[N - c]) / 2 - i W^c (Z[c] - Z*[N - c]) / 2
            const cf p = z[s][4 * (v & 3) + (v >> 2)];
            cf q = zn[s][v];
            if (v == 0 && lane == 0)
                q = p;   // channel 0 is its own partner
            const float er = p.r + q.r, ei = p.i - q.i, dr = p.r - q.r, di = p.i + q.i;
            {
                const float odr = fmaf(wa.r, dr, -(wa.i * di));
                const float odi = v == 0 ? fmaf(wa.r, di, wa.i * dr) : fmaf(wa.i, dr, wa.r * di);
                emit(s, v, false, cf{0.5f * (er + odi), 0.5f * (ei - odr)});
            }
            // the partner's sums and differences are the same up to sign
            // (channel 512 for lane 0, v = 0: its own partner)
            float fr = er, fi = -ei, gr = -dr, gi = di;
            if (v == 0 && lane == 0) {
                const cf m = z[s][2];   // v = 8: u = 0, j2 = 2
                fr = m.r + m.r;
                fi = m.i - m.i;
                gr = m.r - m.r;
                gi = m.i + m.i;
            }
            const float odr = fmaf(wb.r, gr, -(wb.i * gi));
            const float odi = fmaf(wb.i, gr, wb.r * gi);
            emit(s, v, true, cf{0.5f * (fr + odi), 0.5f * (fi - odr)});
        }
    }
}

// LDS: the prototype, the table W2048^c, an exchange buffer per wave and
// (CODES) a code tile per spectrum
// W2048^(l + 64 v) at 2 l + v % 2 of row v / 2 (130 entries); the last two of
// row p serve lane 0's partners: W2048^(64 (2 p + 1)), W2048^(64 (2 p + 2))
// (p = 7: W2048^512)
constexpr int kFeWtEntries = 8 * 130;
constexpr int kFeSmemBase = kFeSmemProto + kFeWtEntries * 8 + kFeWaves * kFeBufFloats * 4;
constexpr int fe_smem_bytes(bool codes, int ns) { return kFeSmemBase + (codes ? ns * kFeN * kFeCodeStride : 0); }

template <bool CODES, int NS>
__device__ __forceinline__ void fengine_body(uint8_t *smem, const FeArgs &a)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // items (NS spectra of an input group g); each XCD takes a contiguous
    // run, so the taps shared by consecutive spectra meet in its L2
    const unsigned groups = a.N / kFeGroup, runs = (a.n_spectra + NS - 1) / NS;
    const unsigned items = runs * groups;
    const unsigned per_xcd = (items + 7) / 8;
    const unsigned first = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const unsigned end = min(items, ((blockIdx.x & 7) + 1) * per_xcd);
    const unsigned stride = gridDim.x >> 3;
    if (first >= end)
        return;

    float4 *hl = (float4 *)smem;
    float2 *wt = (float2 *)(smem + kFeSmemProto);
    float2 *buf = wt + kFeWtEntries + w * (kFeBufFloats / 2);
    uint8_t *codes = smem + kFeSmemBase;

    // the prototype into LDS: float4 (k, t4, l) at (k * 8 + t4) * 64 + l
    for (int idx = threadIdx.x; idx < kFeTaps * 8 * 64; idx += kFeThreads) {
        const int k = idx >> 9, t4 = (idx >> 6) & 7, l = idx & 63;
        hl[idx] = *(const float4 *)(a.h + k * kFeP + 32 * l + 4 * t4);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
        if (v % kFeWaves == w) {
            const cf t = unpack_twiddle(cf{kW2048.re[lane], kW2048.im[lane]}, v);
            const float2 w2 = make_float2(t.r, t.i);
            wt[2 * lane + (v & 1) + 130 * (v >> 1)] = w2;
            if (lane == 0 && v > 0)
                wt[128 + ((v - 1) & 1) + 130 * ((v - 1) >> 1)] = w2;
            if (lane == 0 && v == 8)
                wt[129 + 130 * 7] = w2;
        }
    __syncthreads();

    const FeBases bases{cf{kW1024.re[lane], kW1024.im[lane]}, cf{kW64.re[lane >> 4], kW64.im[lane >> 4]}};
    // this wave's jobs: (item, ii) for items first, first + stride, ... and
    // ii < kFeInputsPerWave; the next job's samples are loaded while the
    // current one is transformed
    FeRaw<NS> raw;
    unsigned run = first % runs, g = first / runs;
    fe_load<NS>(a, g * kFeGroup + w * kFeInputsPerWave, NS * run, raw);
    for (unsigned it = first; it < end; it += stride) {
        const int m = NS * run;
        const unsigned nrun = (it + stride) % runs, ng = (it + stride) / runs;
#pragma unroll 1
        for (int ii = 0; ii < kFeInputsPerWave; ++ii) {
            const int input = g * kFeGroup + w * kFeInputsPerWave + ii;
            cf z[NS][16];
            fe_fir<NS>(raw, hl, z);
            if (ii + 1 < kFeInputsPerWave)
                fe_load<NS>(a, input + 1, m, raw);
            else if (it + stride < end)
                fe_load<NS>(a, ng * kFeGroup + w * kFeInputsPerWave, NS * nrun, raw);
            if constexpr (CODES) {
                // this input's EQ gains, loaded halfway through the transform:
                // late enough to leave its first half the registers, early
                // enough to hide their latency
                const float *gi = a.gains + (int64_t)input * kFeN;
                float g1[8], g2[8];
                auto load_gains = [&]() {
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        g1[v] = gi[lane + 64 * v];
                        g2[v] = gi[v == 0 && lane == 0 ? kFeN / 2 : kFeN - lane - 64 * v];
                    }
                };
                uint8_t *const c1 = codes + lane * kFeCodeStride + w * kFeInputsPerWave + ii;
                uint8_t *const c2 = codes + (kFeN - lane) * kFeCodeStride + w * kFeInputsPerWave + ii;
                uint8_t *const c0 = lane == 0 ? c2 - kFeN / 2 * kFeCodeStride : c2;
                fe_fft<NS>(z, bases, buf, wt, load_gains, [&](int s, int v, bool second, cf y) {
                    // every wave has copied the previous item's codes out
                    // before the first code of this item is written
                    if (s == 0 && v == 0 && !second && ii == 0)
                        lds_barrier();
                    uint8_t *const c = !second ? c1 : v == 0 ? c0 : c2;
                    c[(second ? -64 : 64) * v * kFeCodeStride + s * kFeN * kFeCodeStride] =
                        (uint8_t)pack_code(second ? g2[v] : g1[v], y);
                });
            } else {
                float2 *o = (float2 *)a.out + ((int64_t)input * a.n_spectra + m) * kFeN;
                fe_fft<NS>(z, bases, buf, wt, []() {}, [&](int s, int v, bool second, cf y) {
                    const int c = !second ? lane + 64 * v : v == 0 && lane == 0 ? kFeN / 2 : kFeN - lane - 64 * v;
                    if (m + s < a.n_spectra)
                        o[s * kFeN + c] = make_float2(y.r, y.i);
                });
            }
        }
        if constexpr (CODES) {
            lds_barrier();
            // one 16-byte row per (spectrum, channel): out[m][c][16 g ..]
            // (an opaque thread index: no address kept across the transforms)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            uint8_t *o = (uint8_t *)a.out + ((int64_t)m * kFeN) * a.N + g * kFeGroup;
#pragma unroll
            for (int k = 0; k < NS * kFeN / kFeThreads; ++k) {
                const int c = tid + k * kFeThreads;   // (spectrum, channel)
                const uint32_t *row = (const uint32_t *)(codes + c * kFeCodeStride);
                if (NS == 1 || m + c / kFeN < a.n_spectra)
                    *(uint4 *)(o + (int64_t)c * a.N) = make_uint4(row[0], row[1], row[2], row[3]);
            }
        }
        run = nrun;
        g = ng;
    }
}
#pragma clang fp contract(fast)

template <int NS>
__global__ __launch_bounds__(kFeThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void xc_fengine_kernel(const FeArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[fe_smem_bytes(true, NS)];
    fengine_body<true, NS>(smem, a);
}

template <int NS>
__global__ __launch_bounds__(kFeThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void xc_pfb_spectra_kernel(const FeArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[fe_smem_bytes(false, NS)];
    fengine_body<false, NS>(smem, a);
}

int fe_cu_count()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
        cus = 256;
    return cus;
}

// Persistent grid: kFeWgsPerCu work-groups per compute unit, a multiple of 8
// (one run of items per XCD), no more than there are items per XCD.  Two
// spectra to an item where that takes less time: an item of two costs about 1.6
// of one, and the work-groups take their items in rounds (4112 inputs, one
// spectrum: two rounds either way, 28 us and 41 with two to an item; 192 x 22
// spectra: two rounds and one, 33 and 24).
template <class K1, class K2>
hipError_t fe_launch(K1 one, K2 two, const FeArgs &a, hipStream_t s)
{
    const int cus = fe_cu_count();
    const int64_t groups = a.N / kFeGroup, wgs = cus / 8 * kFeWgsPerCu;   // work-groups per XCD
    const int64_t singles = (a.n_spectra * groups + 7) / 8, pairs = (((int64_t)a.n_spectra + 1) / 2 * groups + 7) / 8;
    const bool both = 8 * ((pairs + wgs - 1) / wgs) < 5 * ((singles + wgs - 1) / wgs);
    const int grid = 8 * (int)std::max<int64_t>(1, std::min(wgs, both ? pairs : singles));
    if (both)
        hipLaunchKernelGGL(two, dim3(grid), dim3(kFeThreads), 0, s, a);
    else
        hipLaunchKernelGGL(one, dim3(grid), dim3(kFeThreads), 0, s, a);
    return hipGetLastError();
}

int fe_check(const void *adc, int64_t S, int32_t N, const float *h, int64_t n_spectra, const void *out)
{
    if (!adc || !h || !out || N < 1 || N % 16 || S < (int64_t)kFeTaps * kFeP || S % 16 ||
        (uintptr_t)adc % 16 || (uintptr_t)h % 16 || (uintptr_t)out % 16 || n_spectra < 1 ||
        n_spectra > S / kFeP - kFeTaps + 1)
        return XCORR_E_INVAL;
    return XCORR_OK;
}

}  // namespace
}  // namespace xc

extern "C" int xcorr_pfb_prototype(int32_t n_points, int32_t taps, float *h_out)
{
    if (n_points < 2 || taps < 1 || !h_out)
        return XCORR_E_INVAL;
    const int64_t L = (int64_t)n_points * taps;
    const double pi = 3.14159265358979323846;
    for (int64_t n = 0; n < L; ++n) {
        const double w = 0.54 - 0.46 * std::cos(2.0 * pi * (double)n / (double)(L - 1));
        const double t = (double)n / n_points - taps / 2.0;
        const double s = t == 0.0 ? 1.0 : std::sin(pi * t) / (pi * t);
        h_out[n] = (float)(w * s);
    }
    return XCORR_OK;
}

extern "C" int xcorr_fengine(const void *d_adc, int64_t n_samples, int32_t n_inputs, const float *d_coeffs,
                             const float *d_gains, int64_t n_spectra, void *d_out, void *stream)
{
    using namespace xc;
    int rc = fe_check(d_adc, n_samples, n_inputs, d_coeffs, n_spectra, d_out);
    if (rc)
        return rc;
    if (!d_gains || (uintptr_t)d_gains % 16)
        return XCORR_E_INVAL;
    const int64_t items = n_spectra * (n_inputs / kFeGroup);
    if (items > (int64_t)1 << 30)
        return XCORR_E_INVAL;
    FeArgs a{(const int8_t *)d_adc, n_samples, n_inputs, d_coeffs, d_gains, (int)n_spectra, d_out};
    const hipError_t e =
        fe_launch(xc_fengine_kernel<1>, xc_fengine_kernel<2>, a, reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? XCORR_OK : api_error(XCORR_E_HIP, std::string("fengine launch: ") + hipGetErrorString(e));
}

extern "C" int xcorr_pfb_spectra(const void *d_adc, int64_t n_samples, int32_t n_inputs, const float *d_coeffs,
                                 int64_t n_spectra, void *d_out, void *stream)
{
    using namespace xc;
    int rc = fe_check(d_adc, n_samples, n_inputs, d_coeffs, n_spectra, d_out);
    if (rc)
        return rc;
    const int64_t items = n_spectra * (n_inputs / kFeGroup);
    if (items > (int64_t)1 << 30)
        return XCORR_E_INVAL;
    FeArgs a{(const int8_t *)d_adc, n_samples, n_inputs, d_coeffs, nullptr, (int)n_spectra, d_out};
    const hipError_t e =
        fe_launch(xc_pfb_spectra_kernel<1>, xc_pfb_spectra_kernel<2>, a, reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? XCORR_OK : api_error(XCORR_E_HIP, std::string("pfb launch: ") + hipGetErrorString(e));
}
