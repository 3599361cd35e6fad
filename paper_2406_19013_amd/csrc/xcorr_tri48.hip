// 4+4-bit int8-MFMA kernel for one triangle of 129 to 192 inputs, on the
// 16 x 16 x 64 form of the matrix instruction.
//
// Arithmetic: the three-product form of xc_gauss4.h, whose scalings, sums and
// bounds hold here as they stand.
//
// Work split.  A persistent work-group of 8 waves, one per compute unit, takes
// the triangle of a channel, cut in four segments of 48 inputs: six waves take
// the 3 x 3 tiles between two segments (27 products per 64 samples), two waves
// the triangles of two segments each (30), so every wave unpacks 6 half blocks
// of 16 inputs, the SIMDs carry 54 or 57 products, and 78 tiles of 16 x 16
// cover what takes 84 in blocks of 32.
//
// Why the 16 x 16 x 64 products: the card runs these kernels at its power limit
// (samples of zeros take 20 % less time for the same cycles), and on the forms'
// operands this instruction sustains 3822 TOP/s, the 32 x 32 x 32 one 3264.
//
// What else it stands on, in the order it was found with cycle counters in the
// kernel: products and unpacking alternate as written; half blocks are unpacked
// in place once their last product is issued, so a wave needs one set of
// operands; the waves of a SIMD raise their priority with each slot and lower
// it as they pass through it, since otherwise the older one runs ahead and
// waits at the barrier for a third of the time (262 -> 256 us); a slot's loads
// are issued between products (issued together after the barrier, each wave
// stood at them for 400 of 3700 cycles); a ring of 4 slots is faster than one
// of 6 (45.1 -> 43.4 us at 192 x 512 x 1024).
//
// Against the three-product kernel on blocks of 32, in one run (cards differ by
// some 5 %): 192 inputs x 1024 channels x 4096 samples 266 -> 250 us (3.8 TB/s);
// 160 x 1024 x 2048 136 -> 127; 192 x 512 x 1024 44.7 -> 42.7; 192 x 4096 x 1024
// 372 -> 367.
#include "xc_mfma4.h"

#include <algorithm>
#include <type_traits>

namespace xc {
namespace {

constexpr int kTsWaves = 8, kTsThreads = 64 * kTsWaves;
constexpr int kTsRows = 128;                        // time rows per ring slot
constexpr int kTsRow = 192;                         // bytes per row
constexpr int kTsSlot = kTsRows * kTsRow;
constexpr int kTsRing = 4;                          // slots
constexpr int kTsLoads = kTsSlot / 1024 / kTsWaves; // 1 KB loads per wave and slot
constexpr int kTsGh = kTsRing * kTsSlot;            // g and h of each input
constexpr int kTsTr = kTsGh + 192 * 8;              // transpose tiles of the two triangle waves
constexpr int kTsSmem = kTsTr + 2 * 16 * 17 * 4;

// 16-byte unit u of time row r lies at u ^ ts_swizzle(r): the 2 x 8 rows of a
// unit that 32 lanes of a transpose read take fall on 64 distinct banks
constexpr int ts_swizzle(int r) { return ((r >> 2) & 1) | ((r >> 4) & 1) << 1; }

// Waves s and s + 4 share a SIMD.  Waves 0..5: the tiles between segments
// row > col; 6, 7: the triangles of segments row and col.
struct TsRole {
    int row, col;
    int sum0, sum1;   // local half blocks whose sums the wave keeps (rows 0..2, columns 3..5; -1: none)
};
constexpr TsRole kTsRoles[8] = {{1, 0, 3, 4}, {2, 0, 0, 5}, {3, 0, 0, 1}, {2, 1, 4, 1},
                                {3, 1, 3, 5}, {3, 2, 5, 2}, {1, 0, -1, -1}, {3, 2, -1, -1}};
constexpr bool ts_triangles(int W) { return W >= 6; }
constexpr int ts_half(int W, int k) { return 3 * (k < 3 ? kTsRoles[W].row : kTsRoles[W].col) + k % 3; }
// tiles: of a pair wave (k / 3, 3 + k % 3); of a triangle wave (0,0) (1,0)
// (1,1) (2,0) (2,1) (2,2) of its rows, then of its columns
constexpr int ts_ntiles(int W) { return ts_triangles(W) ? 12 : 9; }
constexpr int ts_ti(int W, int t) { return ts_triangles(W) ? t / 6 * 3 + tri_I(t % 6) : t / 3; }
constexpr int ts_tj(int W, int t) { return ts_triangles(W) ? t / 6 * 3 + tri_J(t % 6) : 3 + t % 3; }
constexpr bool ts_diag(int W, int t) { return ts_ti(W, t) == ts_tj(W, t); }
struct TsProduct { int t, kind; };
constexpr TsProduct ts_product(int W, int k)   // k-th product: A_i B_j, B_i A_j, R_i R_j tile by tile
{
    for (int t = 0;; ++t)
        for (int kind = 0; kind < 3; ++kind)
            if (!(kind == 1 && ts_diag(W, t)) && k-- == 0)
                return {t, kind};
}

struct TsArgs {
    int64_t T;
    int F, N;
    int per;          // channels per XCD range
    int2 *out;
    const int2 *in;   // running sums (ACC = 1)
};

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

template <int W, int ACC, int MB>
__device__ __forceinline__ void ts_wave(uint8_t *smem, const TsArgs &a, const BlockTable &bt,
                                        const uint8_t *__restrict__ volts)
{
    constexpr int NT = ts_ntiles(W);
    constexpr bool TRI = ts_triangles(W);
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, q = lane & 15;
    lds_u8 *const ring = (lds_u8 *)smem;
    int *const gh = (int *)(smem + kTsGh);

    const int xcd = blockIdx.x & 7, m = (int)(blockIdx.x >> 3), M = gridDim.x >> 3;
    const int first = xcd * a.per;
    const int rlen = min(a.per, a.F - first);
    const int n_my = rlen > m ? (rlen - m + M - 1) / M : 0;
    const int nch = (int)((a.T + kTsRows - 1) / kTsRows);
    const int total = n_my * nch;
    if (total == 0)
        return;
    const int64_t row_bytes = (int64_t)a.F * a.N;
    const uint32_t Tp = (uint32_t)nch * kTsRows;   // samples, with the zero rows of the last slot

    // DMA: load k of this wave fills 64 consecutive units of a slot, whose two
    // halves of 64 rows have a descriptor each (they may lie in two blocks of
    // a table)
    const int half = W >= kTsWaves / 2;
    int is_k = 0, is_c = 0, issued = 0, islot = 0;
    int voff[kTsLoads];
    auto set_item = [&](int k) {
        const int f = first + m + k * M;
        int ln = lane;                        // recomputed per item: kept, these values would take
        asm volatile("" : "+v"(ln));          // the K loop's registers
#pragma unroll
        for (int u = 0; u < kTsLoads; ++u) {
            const int n = 64 * (W * kTsLoads + u) + ln;
            const int r = n / 12;
            const int byte = 16 * ((n % 12) ^ ts_swizzle(r));
            voff[u] = byte < a.N ? (int)((r & 63) * row_bytes) + f * a.N + byte : kBufferOutOfRange;
        }
    };
    set_item(0);
    const uint8_t *src = volts;
    int records = 0;
    lds_u8 *dst = nullptr;
    auto issue_open = [&]() {   // descriptor and ring slot of the stream's next rows
        const int row = is_c * kTsRows + 64 * half;
        const int rows = __builtin_amdgcn_readfirstlane(issued < total ? max(0, min(64, (int)a.T - row)) : 0);
        if constexpr (MB) {
            // addressed from the first block (the restrict-qualified base)
            const int ch = rows > 0 ? row / 64 : 0;
            src = volts + (bt.p[ch / bt.chunks_per_block] - bt.p[0]) +
                  (int64_t)(ch % bt.chunks_per_block) * 64 * row_bytes;
        } else {
            src = volts + (rows > 0 ? row * row_bytes : 0);
        }
        records = __builtin_amdgcn_readfirstlane(rows * (int)row_bytes);
        dst = ring + islot * kTsSlot + W * kTsLoads * 1024;
    };
    auto issue_load = [&](int k) {
        __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc((void *)uniform_pointer(src), (short)0, records, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(dst + k * 1024), 16,
                                                 voff[k], 0, 0, kStreamLoadPolicy);
    };
    auto issue_close = [&]() {
        ++issued;
        islot = islot + 1 == kTsRing ? 0 : islot + 1;
        if (++is_c == nch) {
            is_c = 0;
            if (++is_k < n_my)
                set_item(is_k);
        }
    };

    // operand reads: 16 inputs x 64 samples of a half block; lane: input q,
    // samples 16 g .. 16 g + 15 (read as rows 16 g + (q >> 1) and 8 below)
    const int lane_row = (16 * g + (q >> 1)) * kTsRow + (q & 1) * 8;
    const int swz = ts_swizzle(16 * g + (q >> 1));
    // the swizzle moves a unit within its group of four
    int colo[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        colo[u] = lane_row + ((u ^ swz) << 4);
    v4i X[6];
    auto read = [&](lds_u8 *p, auto kc) {
        constexpr int k = kc, h = ts_half(W, k);
        X[k] = frag_tr8<8 * kTsRow>(p + colo[h & 3] + 64 * (h >> 2));
    };

    v4i A[6], B[6], R[6];
    v4i ab[NT], ba[NT], rr[NT];
    uint32_t sz[2], sl[2];   // sums of the owned half blocks (xc_gauss4.h)
    auto clear = [&]() {
        static_for<0, NT>([&](auto t) { ab[t] = ba[t] = rr[t] = v4i{}; });
        sz[0] = sz[1] = sl[0] = sl[1] = 0;
    };
    clear();
    (void)ba;

    // Instructions at their place in the source: the empty statements keep
    // the compiler from moving them past each other.
    auto product = [&](auto kc) {
        constexpr TsProduct p = ts_product(W, kc);
        constexpr int t = p.t, i = ts_ti(W, t), j = ts_tj(W, t);
        v4i &acc = p.kind == 0 ? ab[t] : p.kind == 1 ? ba[t] : rr[t];
        acc = p.kind == 0   ? __builtin_amdgcn_mfma_i32_16x16x64_i8(A[i], B[j], acc, 0, 0, 0)
              : p.kind == 1 ? __builtin_amdgcn_mfma_i32_16x16x64_i8(B[i], A[j], acc, 0, 0, 0)
                            : __builtin_amdgcn_mfma_i32_16x16x64_i8(R[i], R[j], acc, 0, 0, 0);
        asm volatile("" : "+v"(acc));
    };
    auto unpack = [&](auto kc, auto ec) {   // dword e of half block k
        constexpr int k = kc, e = ec;
        int fa = X[k][e] ^ 0x08080808, fb = X[k][e] ^ 0x07070707, fr = X[k][e] & (int)0xF0F0F0F0;
        asm volatile("" : "+v"(fa), "+v"(fb), "+v"(fr));
        A[k][e] = fa;
        B[k][e] = fb;
        R[k][e] = fr;
    };
    auto sums = [&](auto nc, auto ec) {     // dword e of owned half block n
        constexpr int n = nc, e = ec, k = n ? kTsRoles[W].sum1 : kTsRoles[W].sum0;
        if constexpr (k >= 0) {
            sz[n] = __builtin_amdgcn_sad_u8((uint32_t)(A[k][e] ^ (int)0x80808080), 0u, sz[n]);
            sl[n] = __builtin_amdgcn_sad_u8((uint32_t)A[k][e], (uint32_t)R[k][e], sl[n]);
            asm volatile("" : "+v"(sz[n]), "+v"(sl[n]));
        }
    };
    // Products P0 .. P1 - 1 with `n` pieces of other work spread between
    // them, from the product `lead` on.
    auto products = [&](auto p0, auto p1, auto lead, auto n, auto &&work) {
        constexpr int P0 = p0, NP = p1 - p0, L = lead, N = n;
        static_for<0, NP>([&](auto kc) {
            constexpr int k = kc;
            product(std::integral_constant<int, P0 + k>{});
            if constexpr (k >= L)
                static_for<(k - L) * N / (NP - L), (k - L + 1) * N / (NP - L)>([&](auto u) { work(u); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
#define TS_C(n) std::integral_constant<int, (n)> {}

    auto epilogue = [&](int f) {
        int ln = lane;                        // as in set_item
        asm volatile("" : "+v"(ln));
        // every wave has read the previous channel's g and h
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_no_fence();
        static_for<0, 2>([&](auto nc) {
            constexpr int n = nc, k = n ? kTsRoles[W].sum1 : kTsRoles[W].sum0;
            if constexpr (k >= 0) {
                uint32_t szt = sz[n], slt = sl[n];
                szt += (uint32_t)__shfl_xor((int)szt, 16);
                slt += (uint32_t)__shfl_xor((int)slt, 16);
                szt += (uint32_t)__shfl_xor((int)szt, 32);
                slt += (uint32_t)__shfl_xor((int)slt, 32);
                // g = 16 SR - 15 SA and h = 16 SR - SA, with SR = sum R =
                // szt - slt - 128 Tp and SA = sum A = szt - 128 Tp
                if (ln < 16)
                    *(int2 *)&gh[(16 * ts_half(W, k) + ln) * 2] =
                        make_int2((int)(szt - 16u * slt - 128u * Tp), (int)(15u * szt - 16u * slt - 1920u * Tp));
            }
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_no_fence();
        const int64_t P = (int64_t)a.N * (a.N + 1) / 2;
        const int bytes = (int)(8 * P);
        const int fs = __builtin_amdgcn_readfirstlane(f);
        // rows past input N - 1 lie past the end of the channel's triangle:
        // stores there are dropped, loads give 0
        __amdgpu_buffer_rsrc_t out_f =
            __builtin_amdgcn_make_buffer_rsrc((void *)(a.out + fs * P), (short)0, bytes, 0x00020000);
        __amdgpu_buffer_rsrc_t in_f =
            __builtin_amdgcn_make_buffer_rsrc((void *)(a.in + fs * P), (short)0, bytes, 0x00020000);
        const int jl = ln & 15, il = 4 * (ln >> 4);
        const int part = 4 * il * (il + 1) + 8 * jl, il8 = 8 * il;
        static_for<0, NT / 3>([&](auto sc) {
            // three tiles at a time (registers of the running sums)
            v2i old[ACC ? 12 : 1];
            // byte offset of row r of tile t, 8 (i (i + 1) / 2 + j) for row
            // i = i0 + il + r and column j = j0 + jl, from the lane's part;
            // past the end above the diagonal
            auto offset = [&](auto tc, int r) {
                constexpr int t = tc, i0 = 16 * ts_half(W, ts_ti(W, t)), j0 = 16 * ts_half(W, ts_tj(W, t));
                const int off = part + (i0 + r) * il8 + (4 * (i0 + r) * (i0 + r + 1) + 8 * j0);
                return ts_diag(W, t) && jl > il + r ? kBufferOutOfRange : off;
            };
            if constexpr (ACC)
                static_for<0, 3>([&](auto tt) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        old[4 * tt + r] = __builtin_bit_cast(
                            v2i, __builtin_amdgcn_raw_buffer_load_b64(in_f, offset(TS_C(3 * sc + tt), r), 0, 0));
                });
            static_for<0, 3>([&](auto tt) {
                constexpr int t = 3 * sc + tt;
                constexpr int hi_ = ts_half(W, ts_ti(W, t)), hj = ts_half(W, ts_tj(W, t));
                const v4i g01 = *(const v4i *)&gh[(16 * hi_ + il) * 2], g23 = *(const v4i *)&gh[(16 * hi_ + il + 2) * 2];
                const int2 ghj = *(const int2 *)&gh[(16 * hj + jl) * 2];
                const int gi[4] = {g01.x, g01.z, g23.x, g23.z}, hi[4] = {g01.y, g01.w, g23.y, g23.w};
                const uint32_t ngj = 0u - (uint32_t)ghj.x, hjT = (uint32_t)ghj.y + 128u * Tp;
                v4i bt_;
                if constexpr (ts_diag(W, t)) {
                    int *const tr = (int *)(smem + kTsTr) + (W & 1) * 16 * 17;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        tr[(il + r) * 17 + jl] = ab[t][r];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        bt_[r] = tr[jl * 17 + il + r];
                } else {
                    bt_ = ba[t];
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t pab = (uint32_t)ab[t][r], pba = (uint32_t)bt_[r], prr = (uint32_t)rr[t][r];
                    // 2 Re = 2 P_rr / 256 + 2 Sum im im, P_rr a multiple of 256
                    int imv = (int)(pab + (uint32_t)gi[r] + ngj - pba) >> 5;
                    int re = (int)(2u * prr + (uint32_t)(rr[t][r] >> 7) + (uint32_t)hi[r] + hjT - pab - pba) >> 1;
                    if constexpr (ACC) {
                        re += old[4 * tt + r].x;
                        imv += old[4 * tt + r].y;
                    }
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v2i{re, imv}), out_f,
                                                          offset(TS_C(t), r), 0, 0);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

#pragma unroll
    for (int c = 0; c < kTsRing; ++c) {
        issue_open();
#pragma unroll
        for (int k = 0; k < kTsLoads; ++k)
            issue_load(k);
        issue_close();
    }
    wait_vmcnt_chunks<kTsLoads, kTsRing - 1>(kTsRing - 1);
    barrier_no_fence();
    // operands of a channel's first step
    auto begin = [&](lds_u8 *p) {
        if constexpr (TRI) {
            static_for<0, 6>([&](auto k) { read(p, k); });
            static_for<0, 3>([&](auto k) { static_for<0, 4>([&](auto e) { unpack(k, e); }); });
        } else {
            static_for<0, 6>([&](auto k) { read(p, k); });
            static_for<0, 6>([&](auto k) {
                if constexpr (k != 2 && k != 5)
                    static_for<0, 4>([&](auto e) { unpack(k, e); });
            });
        }
    };
    begin(ring);
    constexpr int STORES = 4 * NT;
    int stored_after = 0;   // slots issued before the last epilogue's stores
    int slot = 0, cc = 0, ck = 0;
    for (int c = 0; c < total; ++c) {
        lds_u8 *const p = ring + slot * kTsSlot;
        slot = slot + 1 == kTsRing ? 0 : slot + 1;
        lds_u8 *const pn = ring + slot * kTsSlot;
        const bool item_end = cc + 1 == nch;
        // The next slot's rows are in LDS when at most what was issued after
        // them is outstanding (memory operations complete in order).  Past
        // the barrier every wave has read all of this slot, which takes the
        // stream's next rows.
        // (Past the stream's end the loads are of no rows.)
        auto next_slot = [&]() {
            if (c + 1 < stored_after)
                wait_vmcnt<(kTsLoads * (kTsRing - 2) + STORES < 63 ? kTsLoads * (kTsRing - 2) + STORES : 63)>();
            else
                wait_vmcnt<kTsLoads * (kTsRing - 2)>();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            barrier_no_fence();
            issue_open();
        };
        // A step of 64 samples.  Half blocks are unpacked in place once their
        // last product of a step is issued (past a channel's or the stream's
        // end what is read and unpacked ahead is not used).
        static_for<0, 2>([&](auto s) {
            lds_u8 *const qn = s ? pn : p + 64 * kTsRow;
            if constexpr (TRI) {
                products(TS_C(0), TS_C(15), TS_C(0), TS_C(12),
                         [&](auto u) { unpack(TS_C(3 + u / 4), TS_C(u % 4)); });
                if constexpr (s)
                    next_slot();
                __builtin_amdgcn_s_setprio(s ? 0 : 2);
                read(qn, TS_C(0));
                read(qn, TS_C(1));
                read(qn, TS_C(2));
                products(TS_C(15), TS_C(30), TS_C(4), TS_C(12), [&](auto u) {
                    unpack(TS_C(u / 4), TS_C(u % 4));
                    if constexpr (s && u % 4 == 0)
                        issue_load(u / 4);
                });
                read(qn, TS_C(3));
                read(qn, TS_C(4));
                read(qn, TS_C(5));
            } else {
                // rows 0, 1, 2: half blocks 0, 1, 2; columns: 3, 4, 5
                products(TS_C(0), TS_C(3), TS_C(0), TS_C(4), [&](auto u) { unpack(TS_C(5), u); });
                products(TS_C(3), TS_C(9), TS_C(0), TS_C(8), [&](auto u) {
                    if constexpr (u % 2 == 0)
                        unpack(TS_C(2), TS_C(u / 2));
                    else
                        sums(TS_C(0), TS_C(u / 2));
                });
                if constexpr (s)
                    next_slot();
                __builtin_amdgcn_s_setprio(s ? 0 : 2);
                read(qn, TS_C(0));
                read(qn, TS_C(1));
                products(TS_C(9), TS_C(18), TS_C(0), TS_C(8), [&](auto u) {
                    if constexpr (u < 4)
                        sums(TS_C(1), u);
                    else
                        unpack(TS_C(0), TS_C(u - 4));
                });
                read(qn, TS_C(3));
                read(qn, TS_C(4));
                if constexpr (s)
                    issue_load(0);
                products(TS_C(18), TS_C(21), TS_C(0), TS_C(4), [&](auto u) { unpack(TS_C(1), u); });
                if constexpr (s)
                    issue_load(1);
                products(TS_C(21), TS_C(24), TS_C(0), TS_C(4), [&](auto u) { unpack(TS_C(3), u); });
                if constexpr (s)
                    issue_load(2);
                products(TS_C(24), TS_C(27), TS_C(0), TS_C(4), [&](auto u) { unpack(TS_C(4), u); });
                read(qn, TS_C(5));
                read(qn, TS_C(2));
            }
            if constexpr (s)
                issue_close();
            __builtin_amdgcn_s_setprio(s ? 3 : 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        ++cc;
        if (item_end) {
            cc = 0;
            epilogue(first + m + ck * M);
            stored_after = issued;
            ++ck;
            clear();
            begin(pn);   // (kept across the epilogue instead: 256 -> 257 us at 192 x 1024 x 4096)
        }
    }
}

template <int ACC, int MB>
__global__ __launch_bounds__(kTsThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void xc_tri48_kernel(const uint8_t *__restrict__ volts, const TsArgs a, const BlockTable bt)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kTsSmem];
    switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: ts_wave<0, ACC, MB>(smem, a, bt, volts); break;
    case 1: ts_wave<1, ACC, MB>(smem, a, bt, volts); break;
    case 2: ts_wave<2, ACC, MB>(smem, a, bt, volts); break;
    case 3: ts_wave<3, ACC, MB>(smem, a, bt, volts); break;
    case 4: ts_wave<4, ACC, MB>(smem, a, bt, volts); break;
    case 5: ts_wave<5, ACC, MB>(smem, a, bt, volts); break;
    case 6: ts_wave<6, ACC, MB>(smem, a, bt, volts); break;
    default: ts_wave<7, ACC, MB>(smem, a, bt, volts); break;
    }
}

}  // namespace

// Measured on both sides of each end (us, this kernel and the one that has the
// work there): 132 inputs x 512 channels x 2048 samples 62 and 76, x 64 channels
// 28 and 30; 192 x 256 x 1024 26.6 and 26.2.  Below 129 inputs the triangles of
// up to four blocks are smaller than its padding; above 192 it has no regions.
// A launch of at most half a slot leaves it behind the three-product kernel
// (192 x 1024 x 64 34.6 and 30.8, x 128 35.7 and 34.1; 160 x 512 x 64 17.3 and
// 15.2; 176 x 4096 x 32 143 and 138), except where it adds to the running sums of
// many channels (144 x 4096 x 64 295 and 310, 192 x 4096 x 32 487 and 498).
bool tri48_taken(int N, int F, int64_t T, bool adds)
{
    return N > 128 && N <= 192 && (T > 64 || (adds && F > 2048));
}

hipError_t launch_tri48(const uint8_t *volts, const BlockTable *bt, int64_t T, int F, int N, int2 *out, const int2 *in,
                        int accumulate, hipStream_t s)
{
    if (T < 1 || T > kMaxSamplesPerLaunch4 || F < 1 || N < 4 || N > 192 || N % 4 || !volts || (uintptr_t)volts % 4 ||
        !out || !in || 64LL * F * N >= (1LL << 31) - 16)
        return hipErrorInvalidValue;
    const TsArgs a{T, F, N, (F + 7) / 8, out, in};
    const int grid = 8 * std::max(1, std::min(compute_units() / 8, a.per));   // one per compute unit
    BlockTable table{};
    if (bt)
        table = *bt;
    auto kern = bt ? (accumulate ? xc_tri48_kernel<1, 1> : xc_tri48_kernel<0, 1>)
                   : (accumulate ? xc_tri48_kernel<1, 0> : xc_tri48_kernel<0, 0>);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kTsThreads), 0, s, volts, a, table);
    return hipGetLastError();
}

}  // namespace xc
