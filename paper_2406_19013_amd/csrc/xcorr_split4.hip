// 4+4-bit int8-MFMA kernel that splits time over the waves of a work-group.
//
// The persistent kernel (xc_gauss4.h) gives a channel's whole triangle to one
// work-group, which walks all of its samples: with fewer channels than
// compute units most of the chip idles.  Here a work-group takes a small
// region of one channel (RB x RB blocks of 32 inputs, on or below the
// diagonal), and its 8 waves take every eighth 32-sample step of it, each
// with a ring of its own, so no wave waits for another before the end, when
// the eight partial sums meet in LDS.
//
// Direct form: R = x & 0xF0 = 16 re and I = (x << 4) & 0xF0 = 16 im are exact
// int8 operands, and R R^T + I I^T = 256 Re, I R^T - R I^T = 256 Im.  On a
// diagonal tile R I^T is the transpose of I R^T.  It costs four products per
// tile (three on the diagonal) where the other kernel's form costs three
// (two), but no per-input sums, which every wave would have to form over its
// share of the samples; padding samples are zero bytes and add nothing.  A
// wave's accumulators hold at most 256 * 128 per sample over an eighth of a
// launch's samples; each partial is a multiple of 256 and is descaled before
// the eight are added.
#include "xc_mfma4.h"

#include <cmath>

namespace xc {
namespace {

constexpr int kSpWaves = 8;
constexpr int kSpThreads = 64 * kSpWaves;
constexpr int kSpStep = 32;            // samples per MFMA K step

// blocks staged, 16-byte units and bytes per time row, LDS-DMA loads and bytes
// per K step
constexpr int sp_blocks(int RB, bool diag) { return diag ? RB : 2 * RB; }
constexpr int sp_units(int RB, bool diag) { return 2 * sp_blocks(RB, diag); }
constexpr int sp_row_bytes(int RB, bool diag) { return 16 * sp_units(RB, diag); }
constexpr int sp_loads(int RB, bool diag) { return sp_units(RB, diag) / 2; }
constexpr int sp_step_bytes(int RB, bool diag) { return kSpStep * sp_row_bytes(RB, diag); }
constexpr int sp_tiles(int RB, bool diag) { return diag ? RB * (RB + 1) / 2 : RB * RB; }
// LDS: the waves' rings (16 KB each for RB = 2, one work-group per CU; 8 KB for
// RB = 1, two), reused for the partial sums of RB tiles at a time (8 waves x
// 2 parts x 4 KB each), and a transpose tile for each
constexpr int kSpTrStride = 33;
constexpr int sp_ring_bytes(int RB) { return RB * 8192; }
constexpr int sp_ring_steps(int RB, bool diag) { return sp_ring_bytes(RB) / sp_step_bytes(RB, diag); }
constexpr int sp_smem_bytes(int RB) { return kSpWaves * sp_ring_bytes(RB) + RB * 32 * kSpTrStride * 4; }
// a 16-byte unit u of time row r lies at u ^ sp_swizzle(r): the 8 rows x 2
// units that two 16-lane groups of a transpose read touch fall on 64 distinct
// banks (rows of 128, 64 and 32 bytes)
constexpr int sp_swizzle(int units, int r) { return units == 8 ? ((r >> 1) & 3) << 1 : units == 4 ? ((r >> 2) & 1) << 1 : 0; }

struct SpArgs {
    int64_t T;        // samples (MB = 1: whole blocks)
    int F, N;
    int nseg;         // segments of RB blocks
    int nreg;         // regions per channel: nseg diagonal ones, then the pairs a > b
    int items;        // F * nreg
    int2 *out;        // [F][P] results
    const int2 *in;   // [F][P] running sums (ACC = 1)
};

__device__ __forceinline__ void sp_wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// One region: rows from segment sa, columns from segment sb (DIAG: sa = sb).
// VEC = 1: rows are 4-byte aligned (N a multiple of 4, 4-byte-aligned input):
// LDS-DMA, whose descriptor ends at the last valid row, so that rows past it
// read as zeros.  VEC = 0: any alignment, staged through registers.  Units
// that reach past input N - 1 bring other channels' inputs into rows and
// columns that are not stored.
template <int RB, bool DIAG, int VEC, int ACC, int MB>
__device__ __forceinline__ void split4_region(uint8_t *smem, const SpArgs &a, const BlockTable &bt,
                                              const uint8_t *__restrict__ volts, int f, int sa, int sb)
{
    constexpr int NB = sp_blocks(RB, DIAG), U = sp_units(RB, DIAG), ROW = sp_row_bytes(RB, DIAG);
    constexpr int NL = sp_loads(RB, DIAG), STEP = sp_step_bytes(RB, DIAG), NBUF = sp_ring_steps(RB, DIAG);
    constexpr int NT = sp_tiles(RB, DIAG), ROWS = 64 / U;   // time rows per load
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, q = lane & 15;
    lds_u8 *const ring = (lds_u8 *)smem + wave * sp_ring_bytes(RB);

    const int64_t row_bytes = (int64_t)a.F * a.N;
    const int nsteps = (int)((a.T + kSpStep - 1) / kSpStep);
    const int mine = nsteps > wave ? (nsteps - wave + kSpWaves - 1) / kSpWaves : 0;

    // staging: load k covers time rows ROWS k .. ROWS k + ROWS - 1; this lane's
    // row within them and byte of the channel's row
    const int lrow = lane / U;
    const int unit = (lane % U) ^ sp_swizzle(U, lrow);
    const int byte = unit < 2 * RB ? 32 * RB * sa + 16 * unit : 32 * RB * sb + 16 * (unit - 2 * RB);
    // operand reads: row (g >> 1) * 16 + (q >> 1) of the step, unit 2 b + (g & 1)
    const int row_off = ((g >> 1) * 16 + (q >> 1)) * ROW + (q & 1) * 8;
    int colo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        colo[b] = ((2 * b + (g & 1)) ^ sp_swizzle(U, q >> 1)) << 4;

    v16i re[NT], im[NT], mi[NT];   // mi: R I^T of an off-diagonal tile
#pragma unroll
    for (int t = 0; t < NT; ++t)
        re[t] = im[t] = mi[t] = v16i{};

    auto row_of = [](int t) { return DIAG ? tri_I(t) : t / RB; };
    auto col_of = [](int t) { return DIAG ? tri_J(t) : t % RB; };
    auto compute = [&](lds_u8 *slot) {
        v4i X[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
            X[b] = frag_tr8<8 * ROW>(slot + row_off + colo[b]);
        return [=, &re, &im, &mi]() {
            v4i R[NB], I[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                R[b] = re16(X[b]);
                I[b] = im16(X[b]);
            }
            static_for<0, NT>([&](auto tc) {
                constexpr int t = tc;
                constexpr int i = DIAG ? tri_I(t) : t / RB, j = DIAG ? tri_J(t) : RB + t % RB;
                re[t] = mfma_i8(R[i], R[j], re[t]);
                im[t] = mfma_i8(I[i], R[j], im[t]);
                if constexpr (!DIAG || i != j)
                    mi[t] = mfma_i8(R[i], I[j], mi[t]);
            });
            static_for<0, NT>([&](auto tc) {
                constexpr int t = tc;
                constexpr int i = DIAG ? tri_I(t) : t / RB, j = DIAG ? tri_J(t) : RB + t % RB;
                re[t] = mfma_i8(I[i], I[j], re[t]);
            });
        };
    };

    if constexpr (VEC) {
        const int voff = byte < a.N ? (int)(lrow * row_bytes) + f * a.N + byte : kBufferOutOfRange;
        int issued = 0, islot = 0;
        auto issue_next = [&]() {
            const int s = wave + issued * kSpWaves;
            const uint8_t *src;
            int64_t left;   // input bytes from the step's first row on
            if constexpr (MB) {
                // addressed from the first block (the restrict-qualified base)
                const int per = 2 * bt.chunks_per_block, blk = s / per, k = s - blk * per;
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
                if (k < mine && t < a.T && byte < a.N) {
                    const uint8_t *const p = volts + t * row_bytes + (int64_t)f * a.N + byte;
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
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
                            x[m] = re[t][4 * rq + m] >> 8;
                            y[m] = (diag ? im[t][4 * rq + m] : im[t][4 * rq + m] - mi[t][4 * rq + m]) >> 8;
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
        int sr[PER], si[PER];
#pragma unroll
        for (int m = 0; m < PER; ++m)
            sr[m] = si[m] = 0;
        if (live) {
            for (int w = 0; w < active; ++w) {
                const lds_v4i *const x = stage + ((su * kSpWaves + w) * 2) * 256 + quad;
                if constexpr (RB == 2) {
                    const v4i p = x[0], v = x[256];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        sr[m] += p[m];
                        si[m] += v[m];
                    }
                } else {
                    const v2i p = *((const lds_v2i_t *)x + (sub >> 1)), v = *((const lds_v2i_t *)(x + 256) + (sub >> 1));
                    sr[0] += p.x;
                    sr[1] += p.y;
                    si[0] += v.x;
                    si[1] += v.y;
                }
            }
        }
        if constexpr (DIAG) {
            // Im of a diagonal tile: I R^T minus its transpose
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
                    int x = sr[m], y = si[m];
                    if constexpr (ACC) {
                        x += old[m].x;
                        y += old[m].y;
                    }
                    out_f[(int64_t)i * (i + 1) / 2 + j] = make_int2(x, y);
                }
            }
        }
    }
}

template <int RB, int VEC, int ACC, int MB>
__global__ __launch_bounds__(kSpThreads) __attribute__((amdgpu_waves_per_eu(RB == 2 ? 2 : 4, RB == 2 ? 2 : 4)))
void xc_split4_kernel(const uint8_t *__restrict__ volts, const SpArgs a, const BlockTable bt)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[sp_smem_bytes(RB)];
    const int item = xcd_item();
    if (item >= a.items)
        return;
    const int f = item / a.nreg, r = item - f * a.nreg;
    if (r < a.nseg) {
        split4_region<RB, true, VEC, ACC, MB>(smem, a, bt, volts, f, r, r);
    } else {
        const int k = r - a.nseg;
        int sa = (int)((1.f + sqrtf(1.f + 8.f * k)) * 0.5f);
        while (sa * (sa - 1) / 2 > k)
            --sa;
        while ((sa + 1) * sa / 2 <= k)
            ++sa;
        split4_region<RB, false, VEC, ACC, MB>(smem, a, bt, volts, f, sa, k - sa * (sa - 1) / 2);
    }
}

template <int RB>
hipError_t split4_launch(const uint8_t *volts, const BlockTable *bt, int64_t T, int F, int N, int2 *out,
                         const int2 *in, int vec, int accumulate, hipStream_t s)
{
    const int nseg = ((N + 31) / 32 + RB - 1) / RB;
    const int64_t nreg = (int64_t)nseg * (nseg + 1) / 2, items = nreg * F;
    if (items > (1LL << 30))
        return hipErrorInvalidValue;
    SpArgs a{T, F, N, nseg, (int)nreg, (int)items, out, in};
    BlockTable table{};
    if (bt)
        table = *bt;
    void (*kern)(const uint8_t *, const SpArgs, const BlockTable);
    if (bt)
        kern = accumulate ? xc_split4_kernel<RB, 1, 1, 1> : xc_split4_kernel<RB, 1, 0, 1>;
    else if (vec)
        kern = accumulate ? xc_split4_kernel<RB, 1, 1, 0> : xc_split4_kernel<RB, 1, 0, 0>;
    else
        kern = accumulate ? xc_split4_kernel<1, 0, 1, 0> : xc_split4_kernel<1, 0, 0, 0>;
    hipLaunchKernelGGL(kern, dim3(xcd_grid((int)items)), dim3(kSpThreads), 0, s, volts, a, table);
    return hipGetLastError();
}

}  // namespace

// Which kernel: estimated times in microseconds, fitted to measurements of
// both kernels over 16 .. 512 inputs, 4 .. 1024 channels and 128 .. 8192
// samples (within about 25 %).  The persistent kernel pays whole rounds of its
// 256 work-groups, each walking every sample; this one pays per work-group
// (512 at a time for regions of one block, 256 for two) plus a part that
// shrinks with the load.  Measured on both sides of the line (this kernel
// against the persistent one): 192 inputs x 4096 samples: 32 channels 20.8 and
// 55 us, 64 channels 37 and 57, 128 channels 55 and 58, 256 channels 109 and
// 69; 64 inputs x 8192: 256 channels 29 and 69, 1024 channels 155 and 138;
// 512 inputs x 8192: 16 channels 84 and 208, 64 channels 301 and 312.  It is
// taken only where the estimate is 10 % better.
int split4_blocks(const Plan &pl, int F, int N, int64_t T)
{
    const double t = (double)T;
    auto regions = [&](int rb) {
        const double nseg = ((N + 31) / 32 + rb - 1) / rb;
        return nseg * (nseg + 1) / 2;
    };
    const double x1 = F * regions(1) / 512.0, x2 = F * regions(2) / 256.0;
    const double one = 3.0 + 2.4 * std::max(1.0, x1) + t * (0.001 + 0.0037 * x1);
    const double two = 3.0 + (4.4 + 0.0034 * t) * std::max(1.0, x2);
    // rounds of the persistent kernel: channel pairs (2 to 4 blocks) or
    // single triangles, then the rectangles of several segments
    const bool pairs = pl.D >= 2 && pl.D <= 4 && F >= 2;
    const double tri = std::ceil((pairs ? (F + 1) / 2 : F) * (double)pl.nseg / 256.0);
    const double rect = std::ceil(F * (double)(pl.regions - pl.nseg) / 256.0);
    const double chunk = pl.D <= 2 ? 0.0078 : pl.D == 3 ? 0.0088 : 0.0117, fixed = pl.D <= 2 ? 3.5 : pl.D == 3 ? 4.5 : 7.0;
    const double persistent = (tri + rect) * (fixed + chunk * t);
    const double best = std::min(one, two);
    return best >= 0.9 * persistent ? 0 : one <= two ? 1 : 2;
}

// Rows off the 4-byte boundaries: the alternative stages every chunk through
// byte loads with two barriers, so this kernel wins (99 inputs x 512 channels:
// 6000 samples 264 against 693 us, 1000 samples 54 against 114) except for a
// few samples of many regions, where the eight partial sums of each tile
// outweigh the products (100 samples: 25 against 23 us).
bool split4_unaligned(int F, int N, int64_t T)
{
    const int64_t nb = (N + 31) / 32, items = nb * (nb + 1) / 2 * F;
    return items <= (1LL << 30) && (T >= 160 || items <= 1024 || nb <= 3);
}

hipError_t launch_split4(int rb, const uint8_t *volts, int64_t T, int F, int N, int2 *acc, int accumulate,
                         hipStream_t s, const int2 *acc_in)
{
    if ((rb != 1 && rb != 2) || T < 1 || T > kMaxSamplesPerLaunch4 || F < 1 || N < 1 || !volts || !acc)
        return hipErrorInvalidValue;
    const int vec = N % 4 == 0 && (uintptr_t)volts % 4 == 0 && 64LL * F * N < (1LL << 31) - 16;
    const int2 *in = acc_in ? acc_in : acc;
    return rb == 2 && vec ? split4_launch<2>(volts, nullptr, T, F, N, acc, in, vec, accumulate, s)
                          : split4_launch<1>(volts, nullptr, T, F, N, acc, in, vec, accumulate, s);
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
    return rb == 2 ? split4_launch<2>(bt.p[0], &bt, T, F, N, acc, acc, 1, accumulate, s)
                   : split4_launch<1>(bt.p[0], &bt, T, F, N, acc, acc, 1, accumulate, s);
}

}  // namespace xc
