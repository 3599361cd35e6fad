// MFMA kernels that split time over the waves of a work-group: 4+4-bit and
// 8+8-bit int8 MFMA, 8+8-bit FP16 MFMA.
//
// The other MFMA kernels give a large region of a channel (up to its whole
// triangle) to one work-group, which walks all of the samples: with fewer
// channels than compute units most of the chip idles.  Here a work-group takes
// a small region of one channel (RB x RB blocks of 32 inputs, on or below the
// diagonal), and its 8 waves take every eighth K step of it, each with a ring
// of its own, so no wave waits for another before the end, when the eight
// partial sums meet in LDS.
//
// 4+4-bit, direct form: R = x & 0xF0 = 16 re and I = (x << 4) & 0xF0 = 16 im are
// exact int8 operands, R R^T + I I^T = 256 Re and I R^T - R I^T = 256 Im.  It
// costs four products per tile (three on the diagonal, where R I^T is the
// transpose of I R^T) where the persistent kernel's form costs three (two),
// but no per-input sums, which every wave would have to form over its share
// of the samples.  A wave's accumulators hold at most 256 * 128 per sample over
// an eighth of a launch's samples; each partial is a multiple of 256 and is
// descaled before the eight are added.
//
// 8+8-bit: samples are (re, im) pairs along K.  X X^T = Re.  int8: with Y = X
// with the bytes of each pair swapped and E = X with the real bytes cleared,
// E_i Y_j^T = sum im_i re_j = P and X_i Y_j^T = P + sum re_i im_j, so Im = 2 P -
// X_i Y_j^T (on the diagonal P - P^T), without negating a byte; wrapping int32
// arithmetic, exact as the final values fit.  FP16: the samples become exact
// halves and Im = X_i X'_j^T with X' = (-im, re).
//
// Padding samples are zero bytes and add nothing in every form.
#include "xc_mfma4.h"

#include <cmath>

namespace xc {
namespace {

constexpr int kSpWaves = 8;
constexpr int kSpThreads = 64 * kSpWaves;

// sample format and arithmetic
constexpr int kSp4 = 0, kSp8 = 1, kSp8H = 2;
constexpr int sp_bytes(int FMT) { return FMT == kSp4 ? 1 : 2; }   // per sample
constexpr int sp_step(int FMT) { return FMT == kSp4 ? 32 : 16; }  // samples per K step (FP16: two MFMA steps)
// blocks staged, 16-byte units and bytes per time row, loads and bytes per K
// step, tiles
constexpr int sp_blocks(int RB, bool diag) { return diag ? RB : 2 * RB; }
constexpr int sp_units(int FMT, int RB, bool diag) { return 2 * sp_bytes(FMT) * sp_blocks(RB, diag); }
constexpr int sp_row_bytes(int FMT, int RB, bool diag) { return 16 * sp_units(FMT, RB, diag); }
constexpr int sp_step_bytes(int FMT, int RB, bool diag) { return sp_step(FMT) * sp_row_bytes(FMT, RB, diag); }
constexpr int sp_loads(int FMT, int RB, bool diag) { return sp_step_bytes(FMT, RB, diag) / 1024; }
constexpr int sp_tiles(int RB, bool diag) { return diag ? RB * (RB + 1) / 2 : RB * RB; }
// LDS: the waves' rings (16 KB each for RB = 2, one work-group per CU; 8 KB for
// RB = 1, two), reused for the partial sums of RB tiles at a time (8 waves x
// 2 parts x 4 KB each), and a transpose tile for each
constexpr int kSpTrStride = 33;
constexpr int sp_ring_bytes(int RB) { return RB * 8192; }
constexpr int sp_ring_steps(int FMT, int RB, bool diag) { return sp_ring_bytes(RB) / sp_step_bytes(FMT, RB, diag); }
constexpr int sp_smem_bytes(int RB) { return kSpWaves * sp_ring_bytes(RB) + RB * 32 * kSpTrStride * 4; }
// A 16-byte unit u of time row r lies at u ^ sp_swizzle(r): what 32 lanes of a
// transpose read touch (4+4-bit: 8 rows x 2 units; 8+8-bit: 4 rows x 4 units)
// falls on 64 distinct banks, for rows of 32 to 256 bytes.
constexpr int sp_swizzle(int FMT, int units, int r)
{
    if (FMT == kSp4)
        return units == 8 ? ((r >> 1) & 3) << 1 : units == 4 ? ((r >> 2) & 1) << 1 : 0;
    return units == 16 ? (r & 3) << 2 : units == 8 ? ((r >> 1) & 1) << 2 : 0;
}

typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v2i sp_tr16(lds_u8 *p)
{
    return __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)p));
}
// two (re, im) byte pairs with the bytes of each pair swapped
__device__ __forceinline__ int sp_swap(int x) { return (int)__builtin_amdgcn_perm((unsigned)x, (unsigned)x, 0x02030001u); }
// two int8 (re, im) pairs -> two half2 (re, im), exact: bytes b + 128 in the
// low mantissa of 1024, less 1152
__device__ __forceinline__ v2i sp_halves(int x)
{
    const unsigned t = (unsigned)x ^ 0x80808080u;
    const unsigned a = __builtin_amdgcn_perm(0x64646464u, t, 0x04010400u);
    const unsigned b = __builtin_amdgcn_perm(0x64646464u, t, 0x04030402u);
    const v2h off = {(_Float16)-1152.0f, (_Float16)-1152.0f};
    return v2i{__builtin_bit_cast(int, __builtin_bit_cast(v2h, a) + off),
               __builtin_bit_cast(int, __builtin_bit_cast(v2h, b) + off)};
}
// half2 (re, im) -> (-im, re)
__device__ __forceinline__ int sp_turn(int h)
{
    return (int)__builtin_amdgcn_alignbit((unsigned)h, (unsigned)h, 16) ^ 0x00008000;
}
__device__ __forceinline__ v16f sp_mfma_f16(v4i a, v4i b, v16f c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}

struct SpArgs {
    int64_t T;        // samples (MB = 1: whole blocks)
    int F, N;
    int nseg;         // segments of RB blocks
    int nreg;         // regions per channel: nseg diagonal ones, then the pairs a > b
    int items;        // F * nreg
    int2 *out;        // [F][P] results (float2 bits for FP16)
    const int2 *in;   // [F][P] running sums (ACC = 1)
};

__device__ __forceinline__ void sp_wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// One region: rows from segment sa, columns from segment sb (DIAG: sa = sb).
// VEC = 1: rows are 4-byte aligned (row bytes and input address multiples of
// 4): LDS-DMA, whose descriptor ends at the last valid row, so that rows past it
// read as zeros.  VEC = 0: any alignment, staged through registers.  Units
// that reach past input N - 1 bring other channels' inputs into rows and
// columns that are not stored.
template <int FMT, int RB, bool DIAG, int VEC, int ACC, int MB>
__device__ __forceinline__ void split_region(uint8_t *smem, const SpArgs &a, const BlockTable &bt,
                                              const uint8_t *__restrict__ volts, int f, int sa, int sb)
{
    constexpr int NB = sp_blocks(RB, DIAG), U = sp_units(FMT, RB, DIAG), ROW = sp_row_bytes(FMT, RB, DIAG);
    constexpr int NL = sp_loads(FMT, RB, DIAG), STEP = sp_step_bytes(FMT, RB, DIAG), NBUF = sp_ring_steps(FMT, RB, DIAG);
    constexpr int NT = sp_tiles(RB, DIAG), ROWS = 64 / U;   // time rows per load
    constexpr int kSpStep = sp_step(FMT), BPS = sp_bytes(FMT), UB = 2 * BPS;   // units per block
    using AccT = typename std::conditional<FMT == kSp8H, v16f, v16i>::type;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, q = lane & 15;
    lds_u8 *const ring = (lds_u8 *)smem + wave * sp_ring_bytes(RB);

    const int64_t row_bytes = (int64_t)a.F * a.N * BPS;
    const int chan_bytes = a.N * BPS;
    const int nsteps = (int)((a.T + kSpStep - 1) / kSpStep);
    const int mine = nsteps > wave ? (nsteps - wave + kSpWaves - 1) / kSpWaves : 0;

    // staging: load k covers time rows ROWS k .. ROWS k + ROWS - 1; this lane's
    // row within them and byte of the channel's row
    const int lrow = lane / U;
    const int unit = (lane % U) ^ sp_swizzle(FMT, U, lrow);
    const int byte = 16 * (unit < UB * RB ? UB * RB * sa + unit : UB * RB * sb + unit - UB * RB);
    // operand reads.  4+4-bit: row (g >> 1) * 16 + (q >> 1) of the step, unit
    // 2 b + (g & 1).  8+8-bit: row (g >> 1) * 8 + (q >> 2) (FP16: 4 instead of 8),
    // unit 4 b + 2 (g & 1) + ((q >> 1) & 1).
    constexpr int GR = FMT == kSp4 ? 16 : FMT == kSp8 ? 8 : 4, QR = FMT == kSp4 ? 1 : 2;
    const int row_off = ((g >> 1) * GR + (q >> QR)) * ROW + (q & 1) * 8;
    int colo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int u = FMT == kSp4 ? 2 * b + (g & 1) : 4 * b + 2 * (g & 1) + ((q >> 1) & 1);
        colo[b] = (u ^ sp_swizzle(FMT, U, q >> QR)) << 4;
    }

    // re: Re's products; im: I R^T, E Y^T (int8) or Im itself (FP16); mi: R I^T
    // or X Y^T of an off-diagonal tile
    AccT re[NT], im[NT], mi[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
        re[t] = im[t] = mi[t] = AccT{};

    auto row_of = [](int t) { return DIAG ? tri_I(t) : t / RB; };
    auto col_of = [](int t) { return DIAG ? tri_J(t) : t % RB; };
    // operands of a step from LDS; the returned call issues its products
    auto compute = [&](lds_u8 *slot) {
        v4i X[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            lds_u8 *const p = slot + row_off + colo[b];
            if constexpr (FMT == kSp4) {
                X[b] = frag_tr8<8 * ROW>(p);
            } else {
                // int8: samples 0..3 and 4..7 of the lane's half; FP16: its 4
                // samples of the first and of the second 8-sample step
                const v2i lo = sp_tr16(p), hi = sp_tr16(p + (FMT == kSp8 ? 4 : 8) * ROW);
                X[b] = v4i{lo.x, lo.y, hi.x, hi.y};
            }
        }
        return [=, &re, &im, &mi]() {
            // products of the first (all tiles), then of the second kind, so
            // that consecutive MFMAs do not share an accumulator
            auto tiles = [&](auto &&f) {
                static_for<0, NT>([&](auto tc) {
                    constexpr int t = tc;
                    f(tc, std::integral_constant<int, DIAG ? tri_I(t) : t / RB>{},
                      std::integral_constant<int, DIAG ? tri_J(t) : RB + t % RB>{});
                });
            };
            if constexpr (FMT == kSp4) {
                v4i R[NB], I[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    R[b] = re16(X[b]);
                    I[b] = im16(X[b]);
                }
                tiles([&](auto t, auto i, auto j) {
                    re[t] = mfma_i8(R[i], R[j], re[t]);
                    im[t] = mfma_i8(I[i], R[j], im[t]);
                    if constexpr (!DIAG || i() != j())
                        mi[t] = mfma_i8(R[i], I[j], mi[t]);
                });
                tiles([&](auto t, auto i, auto j) { re[t] = mfma_i8(I[i], I[j], re[t]); });
            } else if constexpr (FMT == kSp8) {
                v4i E[NB], Y[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    E[b] = X[b] & (int)0xFF00FF00;
                    Y[b] = v4i{sp_swap(X[b].x), sp_swap(X[b].y), sp_swap(X[b].z), sp_swap(X[b].w)};
                }
                tiles([&](auto t, auto i, auto j) {
                    re[t] = mfma_i8(X[i], X[j], re[t]);
                    im[t] = mfma_i8(E[i], Y[j], im[t]);
                    if constexpr (!DIAG || i() != j())
                        mi[t] = mfma_i8(X[i], Y[j], mi[t]);
                });
            } else {
                (void)mi;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    v4i H[NB], T[NB];
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const v2i p = sp_halves(X[b][2 * m]), q = sp_halves(X[b][2 * m + 1]);
                        H[b] = v4i{p.x, p.y, q.x, q.y};
                        T[b] = v4i{sp_turn(p.x), sp_turn(p.y), sp_turn(q.x), sp_turn(q.y)};
                    }
                    tiles([&](auto t, auto i, auto j) {
                        re[t] = sp_mfma_f16(H[i], H[j], re[t]);
                        im[t] = sp_mfma_f16(H[i], T[j], im[t]);
                    });
                }
            }
        };
    };

    if constexpr (VEC) {
        const int voff = byte < chan_bytes ? (int)(lrow * row_bytes) + f * chan_bytes + byte : kBufferOutOfRange;
        int issued = 0, islot = 0;
        auto issue_next = [&]() {
            const int s = wave + issued * kSpWaves;
            const uint8_t *src;
            int64_t left;   // input bytes from the step's first row on
            if constexpr (MB) {
                // addressed from the first block (the restrict-qualified base)
                const int per = 64 / kSpStep * bt.chunks_per_block, blk = s / per, k = s - blk * per;
                src = volts + (bt.p[blk] - bt.p[0]) + (int64_t)k * kSpStep * row_bytes;
                left = (int64_t)(per - k) * kSpStep * row_bytes;
            } else {
                src = volts + (int64_t)s * kSpStep * row_bytes;
                left = (a.T - (int64_t)s * kSpStep) * row_bytes;
            }
            lds_u8 *dst = ring + islot * STEP;
#pragma unroll
            for (int k = 0; k < NL; ++k) {
                const int64_t n = min(left - k * ROWS * row_bytes, ROWS * row_bytes);
                __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(src + k * ROWS * row_bytes), (short)0, n > 0 ? (int)n : 0, 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rsrc, (__attribute__((address_space(3))) void *)(dst + k * 1024), 16, voff, 0, 0, kSharedLoadPolicy);
            }
            ++issued;
            islot = islot + 1 == NBUF ? 0 : islot + 1;
        };
#pragma unroll
        for (int k = 0; k < NBUF; ++k)
            if (k < mine)
                issue_next();
        int slot = 0;
        for (int k = 0; k < mine; ++k) {
            // step k is in LDS when at most the steps issued after it are
            // outstanding (loads complete in order); its slot takes the next
            // step once this wave has its operands
            wait_vmcnt_chunks<NL, NBUF - 1>(issued - 1 - k);
            auto products = compute(ring + slot * STEP);
            sp_wait_lds();
            if (issued < mine)
                issue_next();
            products();
            slot = slot + 1 == NBUF ? 0 : slot + 1;
        }
    } else {
        const uint8_t *const end = volts + a.T * row_bytes;
        v4i st[2][NL];   // the next two steps' units of this lane
        auto load = [&](int k, v4i *v) {
            const int64_t t0 = (int64_t)(wave + k * kSpWaves) * kSpStep + lrow;
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const int64_t t = t0 + u * ROWS;
                v[u] = v4i{0, 0, 0, 0};
                if (k < mine && t < a.T && byte < chan_bytes) {
                    const uint8_t *const p = volts + t * row_bytes + (int64_t)f * chan_bytes + byte;
                    if (p + 16 <= end) {
                        __builtin_memcpy(&v[u], p, 16);   // one unaligned 16-byte load
                    } else {
                        // the last bytes of the input
                        uint32_t w[4] = {0, 0, 0, 0};
                        for (int b = 0; b < 16 && p + b < end; ++b)
                            w[b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
                        v[u] = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
                    }
                }
            }
        };
        typedef __attribute__((address_space(3))) v4i lds_v4i;
        load(0, st[0]);
        load(1, st[1]);
        for (int k = 0; k < mine; k += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (k + h < mine) {
                    // (a wave's LDS accesses execute in order)
                    lds_u8 *const slot = ring + h * STEP;
#pragma unroll
                    for (int u = 0; u < NL; ++u)
                        *(lds_v4i *)(slot + u * 1024 + lane * 16) = st[h][u];
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    auto products = compute(slot);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    load(k + h + 2, st[h]);
                    products();
                }
            }
        }
    }

    // The partial sums of the waves that had samples meet in LDS, RB tiles at
    // a time: a lane's four registers of a row quad are one 16-byte store, and
    // each thread adds a quad (RB = 1: half a quad) of one tile.
    typedef __attribute__((address_space(3))) v4i lds_v4i;
    typedef __attribute__((address_space(3))) v2i lds_v2i_t;
    constexpr int PER = 2 * RB;   // rows of a column per thread
    lds_v4i *const stage = (lds_v4i *)smem;
    int *const tr = (int *)(smem + kSpWaves * sp_ring_bytes(RB));
    const int active = min(kSpWaves, nsteps);
    const int64_t P = (int64_t)a.N * (a.N + 1) / 2;
    int2 *const out_f = a.out + f * P;
    const int2 *const in_f = a.in + f * P;
    // this thread's tile of the round, quad and rows
    const int su = RB == 2 ? threadIdx.x >> 8 : 0, quad = RB == 2 ? threadIdx.x & 255 : threadIdx.x >> 1;
    const int sub = RB == 2 ? 0 : 2 * (threadIdx.x & 1);
    const int r0 = 8 * (quad >> 6) + 4 * ((quad >> 5) & 1) + sub, c0 = quad & 31;   // first row, column in the tile
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += RB) {
        __syncthreads();   // the rings (or the previous round's sums) have been read
        if (wave < active) {
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                const int t = t0 + u;
                if (t < NT) {
                    const bool diag = DIAG && row_of(t) == col_of(t);
#pragma unroll
                    for (int rq = 0; rq < 4; ++rq) {
                        v4i x, y;
                        if constexpr (FMT == kSp8H) {
                            x = __builtin_bit_cast(v4i, v4f{re[t][4 * rq], re[t][4 * rq + 1], re[t][4 * rq + 2],
                                                            re[t][4 * rq + 3]});
                            y = __builtin_bit_cast(v4i, v4f{im[t][4 * rq], im[t][4 * rq + 1], im[t][4 * rq + 2],
                                                            im[t][4 * rq + 3]});
                        } else {
#pragma unroll
                            for (int m = 0; m < 4; ++m) {
                                const int r = 4 * rq + m;
                                if constexpr (FMT == kSp4) {
                                    x[m] = re[t][r] >> 8;
                                    y[m] = (diag ? im[t][r] : im[t][r] - mi[t][r]) >> 8;
                                } else {
                                    x[m] = re[t][r];
                                    y[m] = diag ? im[t][r] : (int)(2u * (uint32_t)im[t][r] - (uint32_t)mi[t][r]);
                                }
                            }
                        }
                        stage[((u * kSpWaves + wave) * 2 + 0) * 256 + rq * 64 + lane] = x;
                        stage[((u * kSpWaves + wave) * 2 + 1) * 256 + rq * 64 + lane] = y;
                    }
                }
            }
        }
        const int t = t0 + su;
        const bool live = t < NT;
        const int ti = row_of(live ? t : 0), tj = col_of(live ? t : 0);
        const bool diag = DIAG && ti == tj;
        const int i0 = (RB * sa + ti) * 32 + r0, j = (RB * sb + tj) * 32 + c0;
        int2 old[PER];
        if constexpr (ACC) {
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const int i = i0 + m;
                const bool ok = live && i < a.N && j <= i;
                old[m] = in_f[ok ? (int64_t)i * (i + 1) / 2 + j : 0];
            }
        }
        __syncthreads();
        using T1 = typename std::conditional<FMT == kSp8H, float, int>::type;
        T1 sr[PER], si[PER];
#pragma unroll
        for (int m = 0; m < PER; ++m)
            sr[m] = si[m] = 0;
        if (live) {
            for (int w = 0; w < active; ++w) {
                const lds_v4i *const x = stage + ((su * kSpWaves + w) * 2) * 256 + quad;
                typedef T1 v4t __attribute__((ext_vector_type(4)));
                typedef T1 v2t __attribute__((ext_vector_type(2)));
                if constexpr (RB == 2) {
                    const v4t p = __builtin_bit_cast(v4t, (v4i)x[0]), v = __builtin_bit_cast(v4t, (v4i)x[256]);
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        sr[m] += p[m];
                        si[m] += v[m];
                    }
                } else {
                    const v2t p = __builtin_bit_cast(v2t, (v2i) * ((const lds_v2i_t *)x + (sub >> 1)));
                    const v2t v = __builtin_bit_cast(v2t, (v2i) * ((const lds_v2i_t *)(x + 256) + (sub >> 1)));
                    sr[0] += p.x;
                    sr[1] += p.y;
                    si[0] += v.x;
                    si[1] += v.y;
                }
            }
        }
        if constexpr (DIAG && FMT != kSp8H) {
            // Im of a diagonal tile: the sum minus its transpose
#pragma unroll
            for (int m = 0; m < PER; ++m)
                tr[su * 32 * kSpTrStride + (r0 + m) * kSpTrStride + c0] = si[m];
            __syncthreads();
            if (diag) {
#pragma unroll
                for (int m = 0; m < PER; ++m)
                    si[m] -= tr[su * 32 * kSpTrStride + c0 * kSpTrStride + r0 + m];
            }
        }
        if (live) {
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const int i = i0 + m;
                if (i < a.N && j <= i) {
                    T1 x = sr[m], y = si[m];
                    if constexpr (ACC) {
                        x += __builtin_bit_cast(T1, old[m].x);
                        y += __builtin_bit_cast(T1, old[m].y);
                    }
                    out_f[(int64_t)i * (i + 1) / 2 + j] =
                        make_int2(__builtin_bit_cast(int, x), __builtin_bit_cast(int, y));
                }
            }
        }
    }
}

template <int FMT, int RB, int VEC, int ACC, int MB>
__global__ __launch_bounds__(kSpThreads) __attribute__((amdgpu_waves_per_eu(RB == 2 ? 2 : 4, RB == 2 ? 2 : 4)))
void xc_split_kernel(const uint8_t *__restrict__ volts, const SpArgs a, const BlockTable bt)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[sp_smem_bytes(RB)];
    const int item = xcd_item(a.items);
    if (item >= a.items)
        return;
    const int f = item / a.nreg, r = item - f * a.nreg;
    if (r < a.nseg) {
        split_region<FMT, RB, true, VEC, ACC, MB>(smem, a, bt, volts, f, r, r);
    } else {
        const int k = r - a.nseg;
        int sa = (int)((1.f + sqrtf(1.f + 8.f * k)) * 0.5f);
        while (sa * (sa - 1) / 2 > k)
            --sa;
        while ((sa + 1) * sa / 2 <= k)
            ++sa;
        split_region<FMT, RB, false, VEC, ACC, MB>(smem, a, bt, volts, f, sa, k - sa * (sa - 1) / 2);
    }
}

template <int FMT, int RB>
hipError_t split_launch(const uint8_t *volts, const BlockTable *bt, int64_t T, int F, int N, void *out,
                        const void *in, int vec, int accumulate, hipStream_t s)
{
    const int nseg = ((N + 31) / 32 + RB - 1) / RB;
    const int64_t nreg = (int64_t)nseg * (nseg + 1) / 2, items = nreg * F;
    if (items > (1LL << 30))
        return hipErrorInvalidValue;
    SpArgs a{T, F, N, nseg, (int)nreg, (int)items, static_cast<int2 *>(out), static_cast<const int2 *>(in)};
    BlockTable table{};
    void (*kern)(const uint8_t *, const SpArgs, const BlockTable);
    if (vec)
        kern = accumulate ? xc_split_kernel<FMT, RB, 1, 1, 0> : xc_split_kernel<FMT, RB, 1, 0, 0>;
    else
        kern = accumulate ? xc_split_kernel<FMT, 1, 0, 1, 0> : xc_split_kernel<FMT, 1, 0, 0, 0>;
    if constexpr (FMT == kSp4)
        if (bt) {
            table = *bt;
            kern = accumulate ? xc_split_kernel<FMT, RB, 1, 1, 1> : xc_split_kernel<FMT, RB, 1, 0, 1>;
        }
    hipLaunchKernelGGL(kern, xcd_grid((int)items), dim3(kSpThreads), 0, s, volts, a, table);
    return hipGetLastError();
}

// rows on 4-byte boundaries, offsets within 64 samples that fit 31 bits
bool split_words(const void *volts, int F, int N, int bps)
{
    return (int64_t)N * bps % 4 == 0 && (uintptr_t)volts % 4 == 0 && 64LL * F * N * bps < (1LL << 31) - 16;
}

}  // namespace

// Which kernel: estimated times in microseconds, fitted to measurements of
// both sides over 16 .. 512 inputs, 4 .. 1024 channels and 128 .. 8192 samples
// (within about 25 %).  The large-region kernels pay whole rounds of 256
// work-groups, each walking every sample; this one pays per work-group (512 at
// a time for regions of one block, 256 for two) plus a part that shrinks with
// the load.  Measured on both sides of the line (this kernel against the
// other): 4+4-bit, 192 inputs: 32 channels x 4096 samples 19 and 48 us, 64 x
// 2048 25 and 29, 128 x 1024 26 and 21; 128 inputs: 64 x 4096 20 and 31, 128 x
// 1024 15 and 12; 256 x 64 x 1024 24 and 30; 384 x 64 x 1024 47 and 34; 512 x 16
// x 2048 33 and 49; 64 inputs x 8192: 256 channels 29 and 69, 1024 channels 155
// and 138; 8+8-bit, 192 inputs x 8192: 32 channels 51 and 138 (FP16 69 and 200),
// 128 channels 142 and 142 (215 and 204); 128 inputs x 128 channels x 4096: 48
// and 47 (63 and 71); FP16 96 x 128 x 4096 61 and 54, 64 x 256 x 8192 57 and 86.
// It is taken only where the estimate is 10 % better.
namespace {
struct SplitCost {
    double one, one_load, two;                   // per sample: one-block regions (base, per load), two-block ones
    double fixed2, fixed3, fixed4, fixed6, rect_fixed;   // the other kernel, a round of D <= 2, 3, 4, 5..6 and of rectangles
    double chunk2, chunk3, chunk4, chunk6, rect_chunk;   // and its time per sample
    bool pairs;                                  // triangles of 2 to 4 blocks go two channels to an item
    bool one_launch;                             // triangles and rectangles fill rounds together
    bool four_bit;                               // arrays that the kernels for 129 .. 192 inputs and for 128-input segments take
};
constexpr SplitCost kCost4{0.001, 0.0037, 0.0034, 3.5, 4.5, 7.0, 7.0, 7.0, 0.0078, 0.0088, 0.0117, 0.0117, 0.0117, true, false, true};
constexpr SplitCost kCost8{0.0015, 0.0062, 0.0052, 2.5, 4.0, 5.0, 9.5, 7.0, 0.0063, 0.0083, 0.0105, 0.0170, 0.0140, false, true, false};
constexpr SplitCost kCost8H{0.0026, 0.006, 0.0072, 3.0, 4.5, 5.0, 9.5, 8.0, 0.0088, 0.0120, 0.0160, 0.0245, 0.0215, false, true, false};

int split_choice(const SplitCost &c, const Plan &pl, int F, int N, int64_t T)
{
    // Up to 256 samples of at most 64 inputs stay with the other kernel.  Measured
    // (us, the other and this one): right for 33 to 64 inputs from 256 channels on
    // (64 x 1024 x 256 11 and 18; 8+8-bit 21 and 20), but this one is the faster
    // below that and for fewer inputs (16 x 8 x 256 5.2 and 3.7 from launch to
    // launch, 32 x 4096 x 256 32 and 22; 8+8-bit 69 and 24).
    if (T <= 256 && pl.D <= 2 && pl.nseg == 1)
        return 0;
    const double t = (double)T;
    auto regions = [&](int rb) {
        const double nseg = ((N + 31) / 32 + rb - 1) / rb;
        return nseg * (nseg + 1) / 2;
    };
    const double x1 = F * regions(1) / 512.0, x2 = F * regions(2) / 256.0;
    const double one = 3.0 + 2.4 * std::max(1.0, x1) + t * (c.one + c.one_load * x1);
    const double two = 3.0 + (4.4 + c.two * t) * std::max(1.0, x2);
    const double fixed = pl.D <= 2 ? c.fixed2 : pl.D == 3 ? c.fixed3 : pl.D == 4 ? c.fixed4 : c.fixed6;
    const double chunk = pl.D <= 2 ? c.chunk2 : pl.D == 3 ? c.chunk3 : pl.D == 4 ? c.chunk4 : c.chunk6;
    const bool pairs = c.pairs && pl.D >= 2 && pl.D <= 4 && F >= 2;
    const double tri_items = (pairs ? (F + 1) / 2 : F) * (double)pl.nseg, rect_items = F * (double)(pl.regions - pl.nseg);
    double other;
    if (c.four_bit && duo4_taken(N, F, T, true)) {
        // two work-groups per compute unit: below half a load a round takes
        // its least time; results are written at about 5 TB/s
        const double nseg = (N + 127) / 128, tri = F * nseg, rect = tri * (nseg - 1) / 2;
        other = 4.5 + t * std::max(0.0068, 0.0168 * tri / 512.0) + 0.0132 * tri;
        if (rect > 0)
            other += 5.7 + t * std::max(0.0115, 0.0185 * rect / 512.0) + 0.026 * rect;
    } else if (c.four_bit && tri48_taken(N, F, T, true)) {
        other = std::ceil(F / 256.0) * (6.0 + 0.0105 * t);
    } else if (c.one_launch && pl.nseg > 1)
        other = std::ceil((tri_items + rect_items) / 256.0) * (c.rect_fixed + c.rect_chunk * t);
    else
        other = std::ceil(tri_items / 256.0) * (fixed + chunk * t) + std::ceil(rect_items / 256.0) * (c.rect_fixed + c.rect_chunk * t);
    return std::min(one, two) >= 0.9 * other ? 0 : one <= two ? 1 : 2;
}

// Rows off the 4-byte boundaries: the alternative stages every chunk through
// byte loads with two barriers, so this kernel wins (99 inputs x 512 channels,
// 4+4-bit: 6000 samples 264 against 693 us, 1000 samples 54 against 114;
// 8+8-bit: 8192 samples 579 against 1886, 128 samples 31 against 40) except for
// a few samples of many regions, where the eight partial sums of each tile
// outweigh the products (4+4-bit, 100 samples: 25 against 23 us).
bool split_any_row(int F, int N, int64_t T, int64_t enough)
{
    const int64_t nb = (N + 31) / 32, items = nb * (nb + 1) / 2 * F;
    return items <= (1LL << 30) && (T >= enough || items <= 1024 || nb <= 3);
}
}  // namespace

// 4+4-bit, arrays whose triangle of 3 to 6 blocks the alternative gives to one
// work-group per channel: it reads the samples once where this kernel reads them
// once per region, so it also wins some hundred samples as long as its rounds of
// 256 work-groups are full (161 inputs, us, this kernel and the other: 160
// samples x 100 channels 14 and 20, x 256 29 and 23, x 300 34 and 41, x 700 70 and
// 62; 450 samples x 256 channels 41 and 42; 65 x 256 x 64 7.9 and 7.1, 65 x 340 x
// 64 9.9 and 12.2).  The estimates are within 10 % of 220 such measurements.
bool split4_unaligned(int F, int N, int64_t T)
{
    if (!split_any_row(F, N, T, 160))
        return false;
    const int nb = (N + 31) / 32;
    if (nb < 3 || nb > 6)
        return true;
    const double t = (double)T, chunks = std::ceil(t / 64), load = std::max(1.0, F * (nb * (nb + 1) / 2) / 512.0);
    const double round = nb == 3   ? 1.65 + 2.35 * chunks + N * (0.0167 + 0.0067 * chunks)
                         : nb == 4 ? 5.1 + 3.0 * chunks
                                   : N * (0.05 + 0.0255 * chunks);
    const double split = 2.4 + 0.005 * t + load * (1.6 + 0.0045 * std::min(t, 300.0) + 0.003 * std::max(0.0, t - 300.0));
    return split < 1.5 + std::ceil(F / 256.0) * round;
}

int split4_blocks(const Plan &pl, int F, int N, int64_t T) { return split_choice(kCost4, pl, F, N, T); }

int split8_blocks(const Plan &pl, bool f16, const uint8_t *volts, int F, int N, int64_t T)
{
    if (split_words(volts, F, N, 2))
        return split_choice(f16 ? kCost8H : kCost8, pl, F, N, T);
    return split_any_row(F, N, T, 128) ? 1 : 0;
}

hipError_t launch_split4(int rb, const uint8_t *volts, int64_t T, int F, int N, int2 *acc, int accumulate,
                         hipStream_t s, const int2 *acc_in)
{
    if ((rb != 1 && rb != 2) || T < 1 || T > kMaxSamplesPerLaunch4 || F < 1 || N < 1 || !volts || !acc)
        return hipErrorInvalidValue;
    const int vec = split_words(volts, F, N, 1);
    const int2 *in = acc_in ? acc_in : acc;
    return rb == 2 && vec ? split_launch<kSp4, 2>(volts, nullptr, T, F, N, acc, in, vec, accumulate, s)
                          : split_launch<kSp4, 1>(volts, nullptr, T, F, N, acc, in, vec, accumulate, s);
}

hipError_t launch_split8(int rb, bool f16, const uint8_t *volts, int64_t T, int F, int N, void *acc,
                         const void *acc_in, int accumulate, hipStream_t s)
{
    if ((rb != 1 && rb != 2) || T < 1 || T > kMaxSamplesPerLaunch8 || F < 1 || N < 1 || !volts || !acc || !acc_in)
        return hipErrorInvalidValue;
    const int vec = split_words(volts, F, N, 2);
    if (f16)
        return rb == 2 && vec ? split_launch<kSp8H, 2>(volts, nullptr, T, F, N, acc, acc_in, vec, accumulate, s)
                              : split_launch<kSp8H, 1>(volts, nullptr, T, F, N, acc, acc_in, vec, accumulate, s);
    return rb == 2 && vec ? split_launch<kSp8, 2>(volts, nullptr, T, F, N, acc, acc_in, vec, accumulate, s)
                          : split_launch<kSp8, 1>(volts, nullptr, T, F, N, acc, acc_in, vec, accumulate, s);
}

hipError_t launch_split4_blocks(int rb, const BlockTable &bt, int n_blocks, int F, int N, int2 *acc, int accumulate,
                                hipStream_t s)
{
    if ((rb != 1 && rb != 2) || n_blocks < 1 || n_blocks > kMaxFusedBlocks || bt.chunks_per_block < 1 ||
        (int64_t)n_blocks * bt.chunks_per_block * 64 > kMaxSamplesPerLaunch4 || F < 1 || N < 1 || N % 16 || !acc ||
        64LL * F * N >= (1LL << 31) - 16)
        return hipErrorInvalidValue;
    for (int b = 0; b < n_blocks; ++b)
        if (!bt.p[b] || (uintptr_t)bt.p[b] % 16)
            return hipErrorInvalidValue;
    const int64_t T = (int64_t)n_blocks * bt.chunks_per_block * 64;
    return rb == 2 ? split_launch<kSp4, 2>(bt.p[0], &bt, T, F, N, acc, acc, 1, accumulate, s)
                   : split_launch<kSp4, 1>(bt.p[0], &bt, T, F, N, acc, acc, 1, accumulate, s);
}

}  // namespace xc
