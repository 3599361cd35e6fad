// 4+4-bit direct-form int8-MFMA kernel with two independent work-groups per
// compute unit, for arrays of 97 to 128 inputs and of several 128-input
// segments.
//
// Work split.  A work-group of 4 waves takes the triangle of a segment, or the
// 4 x 4 blocks between two segments, of one channel; each wave owns tiles of
// its own (a 2 x 2 quarter of a rectangle) over all samples.  Work-groups are
// persistent: each walks its items as one stream through an LDS ring filled by
// LDS-DMA.  Two of them share a compute unit, each with a wave on every SIMD,
// so while one stores its results or waits at its barrier the other's waves
// keep the matrix cores busy; of the 8 waves of one work-group the later on
// each SIMD is always behind, and the earlier waits for it at every barrier.
//
// Arithmetic: R = x & 0xF0 = 16 re and I = (x << 4) & 0xF0 = 16 im; R R^T + I I^T
// = 256 Re and I R^T - R I^T = 256 Im (on a diagonal tile R I^T is the transpose
// of I R^T).  A quarter of a rectangle unpacks 4 blocks for 16 products, 3
// vector instructions per product, which issue beside it (5 do).  The
// three-product form of xc_gauss4.h needs 12, but on operands of 8 significant
// bits, which draw more power, and with 6 instructions and more for each.  An
// accumulator holds at most 256 * 128 per sample, so a launch takes at most
// 65,472 samples.
//
// What bounds it: for a triangle the stream (128 inputs x 2048 channels x 4096
// samples, 1.2 GB: 292 -> 260 us, 4.7 TB/s); for rectangles the power that the
// products draw, then each segment's samples being read once per pair of
// segments.  Against the three-product kernel, in one run: 512 inputs x 512
// channels x 2048 samples 556 -> 474 us; 256 x 512 x 2048 158 -> 136; 1024 x 64 x
// 2048 277 -> 224; and 200 x 512 x 2000 152 -> 125; 128 x 256 x 4096 60 -> 37 (that
// kernel takes channels in pairs, which leaves half the chip idle).
#include "xc_mfma4.h"

#include <algorithm>
#include <type_traits>

namespace xc {
namespace {

constexpr int kDuoTri = 0, kDuoRect = 1;
constexpr int kDuoWaves = 4, kDuoThreads = 64 * kDuoWaves;
constexpr int duo_blocks(int SH) { return SH == kDuoTri ? 4 : 8; }
constexpr int duo_rows(int SH) { return SH == kDuoRect ? 64 : 128; }   // time rows per ring slot
constexpr int duo_row_bytes(int SH) { return 32 * duo_blocks(SH); }
constexpr int duo_slot_bytes(int SH) { return duo_rows(SH) * duo_row_bytes(SH); }
// ring slots of 16 KB (a fourth for rectangles: 139 us for 136 at 256 inputs x
// 512 channels x 2048 samples, nothing elsewhere)
constexpr int kDuoNbuf = 3;
constexpr int kDuoTrStride = 33;                    // ints per row of a transpose tile
constexpr int duo_smem_bytes(int SH)
{
    return kDuoNbuf * duo_slot_bytes(SH) + (SH == kDuoRect ? 0 : 2 * 32 * kDuoTrStride * 4);
}
// 16-byte unit u of time row r lies at u ^ duo_swizzle: the 8 rows x 2 units of
// a transpose read by 32 lanes fall on 64 distinct banks
constexpr int duo_swizzle(int SH, int r)
{
    return SH == kDuoTri ? ((r >> 1) & 3) << 1 : (r & 7) << 1;
}

// Tiles of a wave's role.  Rectangle: quarter (ROLE / 2, ROLE % 2).  Triangle
// of 4 blocks: (0,0) (1,0) (1,1) | (2,2) (3,2) (3,3) | (2,0) (2,1) | (3,0) (3,1).
constexpr int duo_ntiles(int SH, int ROLE) { return SH == kDuoRect ? 4 : ROLE < 2 ? 3 : 2; }
constexpr int duo_row(int SH, int ROLE, int t)
{
    return SH == kDuoRect ? 2 * (ROLE / 2) + t / 2 : ROLE < 2 ? 2 * ROLE + (t > 0) : ROLE;
}
constexpr int duo_col(int SH, int ROLE, int t)   // local block
{
    return SH == kDuoRect ? 4 + 2 * (ROLE % 2) + t % 2 : ROLE < 2 ? 2 * ROLE + (t > 1) : t;
}
constexpr bool duo_uses(int SH, int ROLE, int b)
{
    for (int t = 0; t < duo_ntiles(SH, ROLE); ++t)
        if (duo_row(SH, ROLE, t) == b || duo_col(SH, ROLE, t) == b)
            return true;
    return false;
}
constexpr int duo_nused(int SH, int ROLE)
{
    int n = 0;
    for (int b = 0; b < duo_blocks(SH); ++b)
        n += duo_uses(SH, ROLE, b);
    return n;
}
constexpr int duo_nmfma(int SH, int ROLE)   // products per K step
{
    int n = 0;
    for (int t = 0; t < duo_ntiles(SH, ROLE); ++t)
        n += duo_row(SH, ROLE, t) == duo_col(SH, ROLE, t) ? 3 : 4;
    return n;
}
constexpr int duo_used(int SH, int ROLE, int k)   // the k-th block a role uses
{
    for (int b = 0;; ++b)
        if (duo_uses(SH, ROLE, b) && k-- == 0)
            return b;
}
struct DuoProduct { int t, kind; };
constexpr DuoProduct duo_product(int SH, int ROLE, int k)
{
    for (int t = 0; t < duo_ntiles(SH, ROLE); ++t) {
        const int n = duo_row(SH, ROLE, t) == duo_col(SH, ROLE, t) ? 2 : 3;
        if (k < n)
            return {t, k};
        k -= n;
    }
    return {k, 3};
}
struct DuoArgs {
    int64_t T;        // samples (MB = 1: whole blocks)
    int F, N;
    int nf, lead;     // channels of this launch; bytes of a time row before them
    int ntri, nrect;  // triangles and rectangles per channel
    int2 *out;        // [F][P] results
    const int2 *in;   // [F][P] running sums (ACC = 1)
};

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

// A product at its place in the source: the empty statement keeps the compiler
// from moving it past the unpacking written around it.
__device__ __forceinline__ void fma_in_order(v16i &acc, v4i a, v4i b)
{
    acc = mfma_i8(a, b, acc);
    asm volatile("" : "+v"(acc));
}
__device__ __forceinline__ void unpack_in_order(int x, v4i &re, v4i &im, int e)
{
    int r = x & 0xF0F0F0F0, i = (x << 4) & 0xF0F0F0F0;
    asm volatile("" : "+v"(r), "+v"(i));
    re[e] = r;
    im[e] = i;
}

template <int SH, int ROLE, int ACC, int MB>
__device__ __forceinline__ void duo_wave(uint8_t *smem, const DuoArgs &a, const BlockTable &bt,
                                         const uint8_t *__restrict__ volts, int wave, int nreg)
{
    constexpr int NB = duo_blocks(SH), ROW = duo_row_bytes(SH), SLOT = duo_slot_bytes(SH), NBUF = kDuoNbuf;
    constexpr int C = duo_rows(SH), STEPS = C / 32;
    constexpr int U = 2 * NB;                             // 16-byte units per row
    constexpr int LOADS = SLOT / 1024 / kDuoWaves;            // loads per wave and chunk
    constexpr int NT = duo_ntiles(SH, ROLE);
    const int lane = __lane_id();
    const int g = lane >> 4, q = lane & 15;
    lds_u8 *const ring = (lds_u8 *)smem;

    const int xcd = blockIdx.x & 7, m = (int)(blockIdx.x >> 3), M = gridDim.x >> 3;
    const int per = (a.nf * nreg + 7) / 8;   // this XCD's items (channel, region)
    const int first = xcd * per, rlen = min(per, a.nf * nreg - first);
    const int n_my = rlen > m ? (rlen - m + M - 1) / M : 0;
    const int nch = (int)((a.T + C - 1) / C);
    const int total = n_my * nch;
    if (total == 0)
        return;
    const int64_t row_bytes = (int64_t)a.F * a.N;

    // segments of region k: a triangle's, or the k-th pair sa > sb
    auto segments = [&](int k, int &sa, int &sb) {
        if constexpr (SH == kDuoTri) {
            sa = sb = k;
        } else {
            sa = (int)((1.f + sqrtf(1.f + 8.f * k)) * 0.5f);
            while (sa * (sa - 1) / 2 > k)
                --sa;
            while ((sa + 1) * sa / 2 <= k)
                ++sa;
            sb = k - sa * (sa - 1) / 2;
        }
    };

    // DMA: load k of this wave fills 64 consecutive units of a slot.  A slot of
    // 128 rows is two halves of 64, one per half of the waves, each with a
    // descriptor of its own (the halves may lie in two blocks of a table).
    const int half = C == 128 && wave >= kDuoWaves / 2;
    int is_k = 0, is_c = 0, issued = 0, islot = 0;
    int voff[LOADS];
    auto set_item = [&](int k) {
        const int it = first + m + k * M, f = it / nreg;
        int sa, sb;
        segments(it - f * nreg, sa, sb);
        int ln = __lane_id();                 // recomputed per item: kept, these values would take
        asm volatile("" : "+v"(ln));          // the K loop's registers
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int n = 64 * (wave * LOADS + u) + ln;
            const int r = n / U;
            const int unit = (n % U) ^ duo_swizzle(SH, r);
            const int byte = 16 * unit + (unit < 8 ? 128 * sa : 128 * (sb - 1));
            voff[u] = byte < a.N ? (r & 63) * (int)row_bytes + f * a.N + byte : kBufferOutOfRange;
            __builtin_amdgcn_sched_barrier(0);   // one at a time (registers)
        }
    };
    set_item(0);
    auto issue_next = [&]() {
        const int64_t row = (int64_t)is_c * C + 64 * half;
        const int rows = (int)max((int64_t)0, min((int64_t)64, a.T - row));
        const uint8_t *src;
        if constexpr (MB) {
            // addressed from the first block (the restrict-qualified base)
            const int ch = rows > 0 ? (int)(row / 64) : 0;
            src = volts + (bt.p[ch / bt.chunks_per_block] - bt.p[0]) +
                  (int64_t)(ch % bt.chunks_per_block) * 64 * row_bytes;
        } else {
            src = volts + (rows > 0 ? row * row_bytes : 0);
        }
        __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc((void *)src, (short)0, rows > 0 ? (int)(rows * row_bytes) - a.lead : 0, 0x00020000);
        lds_u8 *dst = ring + islot * SLOT + wave * LOADS * 1024;
#pragma unroll
        for (int k = 0; k < LOADS; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(dst + k * 1024),
                                                     16, voff[k], 0, 0, SH == kDuoRect ? kSharedLoadPolicy : kStreamLoadPolicy);
        ++issued;
        islot = islot + 1 == NBUF ? 0 : islot + 1;
        if (++is_c == nch) {
            is_c = 0;
            if (++is_k < n_my)
                set_item(is_k);
        }
    };

    // operand reads: row (g >> 1) * 16 + (q >> 1) of the K step, unit 2 b + (g & 1)
    const int row_off = ((g >> 1) * 16 + (q >> 1)) * ROW + (q & 1) * 8;
    int colo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        colo[b] = row_off + (((2 * b + (g & 1)) ^ duo_swizzle(SH, q >> 1)) << 4);

    // re: R R^T + I I^T; im: I R^T; mi: R I^T of an off-diagonal tile
    v16i re_[NT], mi_[NT], im[NT];
    auto clear = [&]() {
        static_for<0, NT>([&](auto t) { re_[t] = mi_[t] = im[t] = v16i{}; });
    };
    clear();
    (void)mi_;

    auto read_step = [&](lds_u8 *p, v4i *X) {
        static_for<0, NB>([&](auto b) {
            if constexpr (duo_uses(SH, ROLE, b))
                X[b] = frag_tr8<8 * ROW>(p + colo[b]);
        });
    };
    // unpacked operands: 16x the real and the imaginary parts
    auto unpack = [&](const v4i *X, v4i *R, v4i *I) {
        static_for<0, NB>([&](auto b) {
            if constexpr (duo_uses(SH, ROLE, b)) {
                R[b] = re16(X[b]);
                I[b] = im16(X[b]);
            }
        });
    };
    // Products of a step in issue order: R_i R_j, I_i R_j, R_i I_j of each
    // tile, then the I_i I_j.
    constexpr int NBU = duo_nused(SH, ROLE), NM = duo_nmfma(SH, ROLE);
    auto product = [&](auto kc, const v4i *R, const v4i *I) {
        constexpr DuoProduct d = duo_product(SH, ROLE, kc);
        constexpr int t = d.t, i = duo_row(SH, ROLE, t), j = duo_col(SH, ROLE, t);
        if constexpr (d.kind == 0)
            fma_in_order(re_[t], R[i], R[j]);
        else if constexpr (d.kind == 1)
            fma_in_order(im[t], I[i], R[j]);
        else if constexpr (d.kind == 2)
            fma_in_order(mi_[t], R[i], I[j]);
        else
            fma_in_order(re_[t], I[i], I[j]);
    };
    // A step: its products, with the next step's unpacking spread between
    // them (12 instructions per block, which issue while a product runs).
    auto step = [&](v4i *R, v4i *I, const v4i *X) {
        v4i Rn[NB], In[NB];
        static_for<0, NM>([&](auto k) {
            product(k, R, I);
            static_for<k * 4 * NBU / NM, (k + 1) * 4 * NBU / NM>([&](auto u) {
                constexpr int b = duo_used(SH, ROLE, u / 4), e = u % 4;
                unpack_in_order(X[b][e], Rn[b], In[b], e);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<0, NB>([&](auto b) {
            if constexpr (duo_uses(SH, ROLE, b)) {
                R[b] = Rn[b];
                I[b] = In[b];
            }
        });
    };
    // A rectangle's accumulators leave no registers for a second set of
    // operands, but a block is dead once its tiles are done: tile by tile,
    // the block that the next tile but one needs is unpacked in its place.
    auto phase = [&](auto tc, auto bc, v4i *R, v4i *I, const v4i *X) {
        constexpr int t = tc, b = bc, i = duo_row(SH, ROLE, t), j = duo_col(SH, ROLE, t);
        static_for<0, 4>([&](auto k) {
            if constexpr (k == 0)
                fma_in_order(re_[t], R[i], R[j]);
            else if constexpr (k == 1)
                fma_in_order(im[t], I[i], R[j]);
            else if constexpr (k == 2)
                fma_in_order(mi_[t], R[i], I[j]);
            else
                fma_in_order(re_[t], I[i], I[j]);
            constexpr int e = k;
            unpack_in_order(X[b][e], R[b], I[b], e);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    auto epilogue = [&](int it) {
        const int f = __builtin_amdgcn_readfirstlane(it / nreg);
        int sa, sb;
        segments(it - f * nreg, sa, sb);
        const int64_t P = (int64_t)a.N * (a.N + 1) / 2;
        const int bytes = (int)(8 * P);
        // rows past input N - 1 lie past the end of the channel's triangle:
        // stores there are dropped, loads give 0
        __amdgpu_buffer_rsrc_t out_f =
            __builtin_amdgcn_make_buffer_rsrc((void *)(a.out + f * P), (short)0, bytes, 0x00020000);
        __amdgpu_buffer_rsrc_t in_f =
            __builtin_amdgcn_make_buffer_rsrc((void *)(a.in + f * P), (short)0, bytes, 0x00020000);
        int ln = __lane_id();                 // as in set_item
        asm volatile("" : "+v"(ln));
        const int jl = ln & 31, il0 = 4 * (ln >> 5);
        static_for<0, NT>([&](auto tc) {
            constexpr int t = tc, I = duo_row(SH, ROLE, t), J = duo_col(SH, ROLE, t);
            constexpr bool diag = I == J;
            const int i0 = (4 * sa + I) * 32 + il0, j = (4 * sb + (SH == kDuoRect ? J - 4 : J)) * 32 + jl;
            auto offset = [&](int r) {
                const int i = i0 + 8 * (r >> 2);
                const int u = r & 3;
                const int off = 4 * (int)__umul24(i, i + 1) + 8 * j + u * (8 * i) + 4 * u * (u + 1);
                return diag && j > i + u ? kBufferOutOfRange : off;
            };
            // running sums, OR rows at a time (registers)
            constexpr int OR = SH == kDuoRect ? 4 : 16;
            v2i old[ACC ? OR : 1];
            auto load_old = [&](int r0) {
#pragma unroll
                for (int r = 0; r < OR; ++r)
                    old[r] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(in_f, offset(r0 + r), 0, 0));
            };
            if constexpr (ACC)
                load_old(0);
            v16i mi;
            if constexpr (diag) {
                int *const tr = (int *)(smem + NBUF * SLOT) + ROLE * 32 * kDuoTrStride;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    tr[(8 * (r >> 2) + il0 + (r & 3)) * kDuoTrStride + jl] = im[t][r];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    mi[r] = tr[jl * kDuoTrStride + 8 * (r >> 2) + il0 + (r & 3)];
            } else {
                mi = mi_[t];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int re = re_[t][r] >> 8, imv = (im[t][r] - mi[r]) >> 8;
                if constexpr (ACC) {
                    if (r > 0 && r % OR == 0) {
                        __builtin_amdgcn_sched_barrier(0);
                        load_old(r);
                    }
                    re += old[r % OR].x;
                    imv += old[r % OR].y;
                }
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v2i{re, imv}), out_f, offset(r), 0, 0);
            }
            if constexpr (ACC)
                __builtin_amdgcn_sched_barrier(0);
        });
    };

#pragma unroll
    for (int c = 0; c < NBUF; ++c)
        if (c < total)
            issue_next();
    wait_vmcnt_chunks<LOADS, NBUF - 1>(issued - 1);
    barrier_no_fence();
    constexpr bool AHEAD = SH != kDuoRect;
    v4i X[NB], R[NB], I[NB];   // packed operands read ahead, unpacked ones of the current step
    // blocks of a rectangle role: rows b0, b1, columns c0, c1
    constexpr auto kB0 = std::integral_constant<int, duo_row(SH, ROLE, 0)>{};
    constexpr auto kC0 = std::integral_constant<int, duo_col(SH, ROLE, 0)>{};
    constexpr auto kB1 = std::integral_constant<int, AHEAD ? 0 : kB0 + 1>{};
    constexpr auto kC1 = std::integral_constant<int, AHEAD ? 0 : kC0 + 1>{};
    auto read = [&](lds_u8 *p, int b) { X[b] = frag_tr8<8 * ROW>(p + colo[b]); };
    // operands of an item's first step
    auto begin = [&](lds_u8 *p) {
        if constexpr (AHEAD) {
            read_step(p, X);
            unpack(X, R, I);
            read_step(p + 32 * ROW, X);
        } else {
            read(p, kB0);
            read(p, kC0);
            read(p, kC1);
            R[kB0] = re16(X[kB0]);
            I[kB0] = im16(X[kB0]);
            R[kC0] = re16(X[kC0]);
            I[kC0] = im16(X[kC0]);
        }
    };
    begin(ring);
    constexpr int STORES = 16 * NT;
    int stored_after = 0;   // chunks issued before the last epilogue's stores
    int slot = 0, cc = 0, ck = 0;
    for (int c = 0; c < total; ++c) {
        lds_u8 *const p = ring + slot * SLOT;
        slot = slot + 1 == NBUF ? 0 : slot + 1;
        lds_u8 *const pn = ring + slot * SLOT;
        const bool more = c + 1 < total, item_end = cc + 1 == nch;
        // The next chunk is in LDS when at most what was issued after it is
        // outstanding (memory operations complete in order).  Past the
        // barrier every wave has read all of this chunk, whose slot takes the
        // stream's next chunk.
        auto next_chunk = [&]() {
            if (more) {
                const int r = issued - 2 - c;
                if (c + 1 < stored_after)
                    wait_vmcnt_chunks_after<LOADS, NBUF - 1, STORES>(r);
                else
                    wait_vmcnt_chunks<LOADS, NBUF - 1>(r);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                barrier_no_fence();
                if (issued < total)
                    issue_next();
            }
        };
        // (past an item's or the stream's end the reads ahead are of data not
        // used)
        if constexpr (AHEAD) {
            static_for<0, STEPS - 2>([&](auto s) {
                step(R, I, X);
                read_step(p + (s + 2) * 32 * ROW, X);
                __builtin_amdgcn_sched_barrier(0);
            });
            step(R, I, X);
            next_chunk();
            read_step(pn, X);
            __builtin_amdgcn_sched_barrier(0);
            step(R, I, X);
            read_step(pn + 32 * ROW, X);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            constexpr std::integral_constant<int, 0> k0{};
            constexpr std::integral_constant<int, 1> k1{};
            constexpr std::integral_constant<int, 2> k2{};
            constexpr std::integral_constant<int, 3> k3{};
            static_for<0, STEPS>([&](auto sc) {
                constexpr int s = sc;
                read(p + s * 32 * ROW, kB1);
                phase(k0, kC1, R, I, X);
                if constexpr (s + 1 == STEPS)
                    next_chunk();
                lds_u8 *const q = s + 1 == STEPS ? pn : p + (s + 1) * 32 * ROW;
                read(q, kB0);
                phase(k1, kB1, R, I, X);
                read(q, kC0);
                phase(k2, kB0, R, I, X);
                read(q, kC1);
                phase(k3, kC0, R, I, X);
            });
        }
        ++cc;
        if (item_end) {
            cc = 0;
            epilogue(first + m + ck * M);
            stored_after = issued;
            ++ck;
            clear();
            begin(pn);
        }
    }
}

template <int SH, int ACC, int MB>
__device__ __forceinline__ void duo_roles(uint8_t *smem, const DuoArgs &a, const BlockTable &bt,
                                          const uint8_t *__restrict__ volts, int wave, int nreg)
{
    // two work-groups' waves of one SIMD take different roles (a triangle's
    // roles carry 10 and 8 products)
    switch ((wave + 2 * ((blockIdx.x >> 3) & 1)) & 3) {
    case 0: duo_wave<SH, 0, ACC, MB>(smem, a, bt, volts, wave, nreg); break;
    case 1: duo_wave<SH, 1, ACC, MB>(smem, a, bt, volts, wave, nreg); break;
    case 2: duo_wave<SH, 2, ACC, MB>(smem, a, bt, volts, wave, nreg); break;
    default: duo_wave<SH, 3, ACC, MB>(smem, a, bt, volts, wave, nreg); break;
    }
}

// Every work-group walks its share of the triangles and of the rectangles, the
// first half of an XCD's work-groups the triangles first, the second half, which
// joins them on the compute units, the rectangles first: the triangles' stream
// and the rectangles' products then share the chip.  One launch for each shape
// took 500 us at 512 inputs x 512 channels x 2048 samples, this 486 beside it; 256 x 512 x
// 2048 150 and 137; 384 x 64 x 1024 35 and 32.
template <int ACC, int MB>
__global__ __launch_bounds__(kDuoThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void xc_duo4_kernel(const uint8_t *__restrict__ volts, const DuoArgs a, const BlockTable bt)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[duo_smem_bytes(kDuoTri) > duo_smem_bytes(kDuoRect)
                                                               ? duo_smem_bytes(kDuoTri) : duo_smem_bytes(kDuoRect)];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool rect_first = (blockIdx.x >> 3) >= (gridDim.x >> 4);
    for (int k = 0; k < 2; ++k) {
        if (rect_first == (k == 0)) {
            if (a.nrect)
                duo_roles<kDuoRect, ACC, MB>(smem, a, bt, volts, wave, a.nrect);
        } else {
            duo_roles<kDuoTri, ACC, MB>(smem, a, bt, volts, wave, a.ntri);
        }
        __syncthreads();   // the ring and the transpose tiles change hands
    }
}

}  // namespace

// Where neither a single triangle of up to three blocks nor the kernel for one
// of 129 to 192 inputs does the work.  Measured at both ends against the
// three-product kernel (us): 100 inputs x 256 channels x 2048 samples 20 and
// 34; 128 x 512 x 4096 69 and 71; 200 x 16 x 2048 47 and 60; 2048 x 8 x 512 49
// and 61; 300 x 512 x 64 46 and 51; 128 x 1024 x 64 16.2 and 17.0.  With 96 inputs a
// quarter of the triangle would be padding.  One triangle of up to 112 inputs,
// many channels and a few samples is all epilogue, which the other kernel has
// the shorter of where nothing is added to running sums (112 x 4096 x 64 48.4 and
// 41.5, adding 170 and 179; 128 x 4096 x 32 53.1 and 51.3, but 234 and 239 with a
// second launch that adds to it).
bool duo4_taken(int N, int F, int64_t T, bool adds)
{
    if (T > kMaxSamplesDuo4)
        return false;
    return N > 192 || (N > 96 && N <= 128 && (adds || N > 112 || T > 64 || F <= 2048));
}

// A launch of more than about 2 ms goes as two, each over half of the channels:
// its work-groups hold every compute unit to its end, and another stream's
// kernel waits for that.  96, 192 and 512 inputs x 4096 channels streaming side
// by side: the 192-input array's p99 per block of 1024 samples 4.13 -> 2.28 ms
// (2.98 when triangles and rectangles were a launch each), per group of 8 blocks
// 19.3 -> 10.8 (15.3); the 512-input array's 4.19 -> 4.54 (4.62) and 19.4 -> 21.3
// (23.2).  By itself the 512-input launch gains, as fewer channels are under way
// at once (3410 -> 3375 us, 8 blocks 16,300 -> 15,700).
static int duo4_launches(int64_t T, int F, int regions) { return F > 1 && T * F * regions >= 30000000 ? 2 : 1; }

hipError_t launch_duo4(const uint8_t *volts, const BlockTable *bt, int64_t T, int F, int N, int2 *out, const int2 *in,
                       int accumulate, hipStream_t s)
{
    if (T < 1 || T > kMaxSamplesDuo4 || F < 1 || N < 4 || N % 4 || !volts || (uintptr_t)volts % 4 || !out || !in ||
        64LL * F * N >= (1LL << 31) - 16)
        return hipErrorInvalidValue;
    const int nseg = (N + 127) / 128, pairs = nseg * (nseg - 1) / 2;
    if ((int64_t)F * std::max(nseg, pairs) > (1LL << 30))
        return hipErrorInvalidValue;
    BlockTable table{};
    if (bt)
        table = *bt;
    auto kern = bt ? (accumulate ? xc_duo4_kernel<1, 1> : xc_duo4_kernel<0, 1>)
                   : (accumulate ? xc_duo4_kernel<1, 0> : xc_duo4_kernel<0, 0>);
    const int launches = duo4_launches(T, F, nseg + pairs);
    for (int k = 0; k < launches; ++k) {
        const int f0 = (int)((int64_t)F * k / launches), nf = (int)((int64_t)F * (k + 1) / launches) - f0;
        const int64_t P = (int64_t)N * (N + 1) / 2;
        const DuoArgs a{T, F, N, nf, f0 * N, nseg, pairs, out + f0 * P, in + f0 * P};
        const int per = (int)(((int64_t)nf * std::max(nseg, pairs) + 7) / 8);
        const int grid = 8 * std::max(1, std::min(compute_units() / 4, per));   // two per compute unit
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kDuoThreads), 0, s, volts + (int64_t)f0 * N, a, table);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace xc
