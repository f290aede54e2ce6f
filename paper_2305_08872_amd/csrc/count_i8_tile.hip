// Join count on the int8 matrix cores for operands of any size, alignment and layout, in place.
//
// A workgroup owns a tile of 256 x 256, 192 x 256, 128 x 256, 128 x 128 or 64 x 64 counts (the last with two groups of
// waves that share K) and walks K in stages of 64: v_mfma_i32_32x32x32_i8 on fragments that an operand stored
// along k gives by ds_read_b128 and one stored across k by ds_read_b64_tr_b8, which transposes on the way.  So
// the four layouts are four kernels of one body, and none is copied first.  What bounds it: at large sizes the
// matrix cores and, one workgroup per unit or two that run in step, the write-back of the tile that they
// wait for; at small ones the start of a launch and the first loads (1000^3 6.5 us, of which the matrix cores
// are busy 1.2).
//
// Edges cost no pass and no copy: a line past the edge reads the last one inside it; a 16-byte unit that would
// cross the end of a line across k reads the last 16 bytes inside and its place in the tile moves with it
// (row_of / col_of: every count is written from one place); the last, short stage of a k range is the 64 k that
// end at K, with A's bytes already summed zeroed.  Every access stays inside the operands.
//
// Two ways in.  Streamed (global_load_lds, a ring of 3 or 4 stages; the 128 x 256 tile, alone on its unit, of 6:
// 2048 x 4096 x 4096 49 -> 36 us, while the smaller tiles gain nothing from 8) where pieces of rows start at 4-byte
// addresses: 64 KiB in flight per unit and no register or LDS-write cycles.  Through registers (two sets, two
// LDS slots) for rows at any byte address, 42-67 % more per stage by tile; a whole call, us, streamed / the same
// call one byte off: 3000 x 4004 x 2504 (written) 38 / 49, 5000 x 7000 x 3000 145 / 175, 8000^2 x 4000 235 / 314,
// 2048^2 x 8192 40 / 67.
//
// With at most one workgroup to a unit the smaller tiles take stages of 128 k (a ring of 4, 128 KiB): half the barriers, twice the bytes in
// flight and, of lines along k, whole lines of the caches at a time. us, stages of 64 k / of 128, calls on three sets of matrices in turn:
// 1024^2 x 4096 14.6 / 13.3, 2048^3 15.9 / 14.8, 1536^2 x 8192 36.8 / 32.3, 2412 x 896 x 4184 27.0 / 23.6, 320 x 2688 x
// 7808 22.4 / 19.6, 288 x 7744 x 3968 23.2 / 19.6, 448 x 5012 x 5040 with B transposed 33.9 / 29.2.  Two workgroups to a unit have no room for it.
// (Through registers the same, with one set of registers: 4 us more at the start and 4 % less per k, 2999 x 4001 x 2503 39.6 / 43.6.)
//
// Through registers a stage takes 0.8 us in a tile of 256 rows and in one of 192 (not its loads' round trip: with 4 stages on their
// way in registers instead of 2 the same), and what a unit does not overlap is the write-back of its tile, 24 us and 19: so rows at any
// address have a tile of 192 x 256, us, 256 / 192: 2999 x 4001 x 2503 57.7 / 53.3 (written 52 / 47), 6000 x 6001 x 1501 113 / 100,
// 5999 x 4001 x 2503 104 / 94, with B transposed 110 / 101, 3071 x 4095 x 8191 127 / 121.
//
// Measured, us, the kernels it replaced at these sizes / here: 1000^3 38 / 6.5 (a stage of 128 x 128 guarded
// loads by one thread each), 2999 x 4001 x 2503 (written) 79 / 45, 5000 x 7000 x 3000 212 / 145, 8191^2 x 4095
// 562 / 314, 8000^2 x 4000 368 / 235, 2048^2 x 8192 57 / 40; 4096^3 with both operands transposed 85 / 64.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amulet_internal.h"

// the LDS-DMA asm below sets M0 itself and says so in its clobber list
#pragma clang diagnostic ignored "-Winline-asm"

namespace amulet {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef v4i v4i_any __attribute__((aligned(1)));
typedef v4i v4i_r __attribute__((aligned(4)));
typedef __attribute__((address_space(3))) v2i *lds_v2i_ptr;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

extern __shared__ __attribute__((aligned(16))) int8_t ct_smem[];

constexpr int CT_BK = 64;

template <int N> __device__ __forceinline__ void ct_wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// resident waves per SIMD the registers are held to (the workgroup of 12 waves has its unit for itself)
constexpr int ct_waves(int waves) { return waves == 12 ? 3 : 4; }

// Waves: WK groups of WR x WC, a group sums its own kgroup of the workgroup's k; a wave MB x NB blocks of 32 x 32.
// NST: stages of the ring.  TA / TB: A stored K x M / B stored N x K.  REG: through registers.  KS: K over several workgroups.
// NT: R is read and written around the caches.
// BK: k of a stage, 64 or (streamed only) 128.
template <int MB, int NB, int WR, int WC, int WK, int NST, bool TA, bool TB, bool REG, bool KS, bool NT, int BK>
__global__ void __launch_bounds__(64 * WR * WC * WK) __attribute__((amdgpu_waves_per_eu(ct_waves(WR * WC * WK), ct_waves(WR * WC * WK))))
count_i8_tile_kernel(const CountTileArgs args)
{
    constexpr int BM = 32 * MB * WR, BN = 32 * NB * WC;
    constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, G_BYTES = A_BYTES + B_BYTES, STAGE_BYTES = WK * G_BYTES;
    constexpr int NW = WR * WC;                          // waves of a group
    constexpr int LINES = G_BYTES / 1024, A_LINES = A_BYTES / 1024, LOADS = (LINES + NW - 1) / NW;
    constexpr int A_LOADS = A_LINES / NW;                // of a wave's loads the first ones are A's
    constexpr bool RAGGED = LINES % NW != 0;             // the last load is the first waves' only
    static_assert((REG || !RAGGED) && A_LINES % NW == 0, "the stage's kilobytes divide over the group's waves");
    static_assert(!(TA && (BM & (BM - 1)) != 0), "the units of a k-row are exchanged within powers of two");
    static_assert(BK == 64 || (BK == 128 && !REG), "stages of 64 k, streamed ones also of 128");
    constexpr int UK = BK / 16;                          // 16-byte units of a line along k
    constexpr int UA = BM / 16, UB = BN / 16;            // 16-byte units in a k-row of an operand kept k-major

    const int M = args.M, N = args.N, K = args.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = wave / NW, wg = wave % NW, wr = wg / WC, wc = wg % WC;
    const int li = lane & 31, lh = lane >> 5;

    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, (M + BM - 1) / BM, (N + BN - 1) / BN, tm, tn)) return;
    const int row0 = __builtin_amdgcn_readfirstlane(tm * BM), col0 = __builtin_amdgcn_readfirstlane(tn * BN);
    const int part0 = (int)blockIdx.y * args.kpart;
    const int part_len = K - part0 < args.kpart ? K - part0 : args.kpart;
    const int kb = part0 + g * args.kgroup;
    int klen = part_len - g * args.kgroup;
    klen = klen < 0 ? 0 : klen < args.kgroup ? klen : args.kgroup;
    const int n_full = klen / BK, tail = klen - n_full * BK;
    const int n_st = ((args.kgroup < part_len ? args.kgroup : part_len) + BK - 1) / BK;

    // unit u of line r of an operand kept k-minor stands at u ^ along(r), unit u of k-row k of one kept k-major at u ^ swz(k)
    auto along = [](int r) { return UK == 4 ? (r >> 2) & 3 : (r >> 1) & 7; };
    auto swz = [](int units, int k) { return 2 * (((k & 7) / (16 / units)) & (units / 2 - 1)); };

    const int rbase = TA && row0 > M - 16 ? M - 16 : row0, cbase = !TB && col0 > N - 16 ? N - 16 : col0;
    uint32_t voff[LOADS];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_ptr)ct_smem;
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
        const int line = !RAGGED || q < LOADS - 1 || wg + NW * q < LINES ? wg + NW * q : wg + NW * (q - 1);
        const bool is_a = q < A_LOADS;
        const int s = (is_a ? line : line - A_LINES) * 64 + lane;
        const int edge = is_a ? M : N, org = is_a ? row0 : col0, base = is_a ? rbase : cbase;
        const uint32_t ld = (uint32_t)(is_a ? args.lda : args.ldb);
        if (is_a ? !TA : TB) {       // lines along k: BK bytes each
            const int r = s / UK, u = (s % UK) ^ along(r);
            const int rc = org + r < edge ? r : edge - 1 - org;
            voff[q] = (uint32_t)rc * ld + (uint32_t)(u * 16);
        } else {
            const int units = is_a ? UA : UB;
            const int k = s / units, u = (s % units) ^ swz(units, k);
            const int start = org + u * 16 < edge - 16 ? org + u * 16 : edge - 16;
            voff[q] = (uint32_t)k * ld + (uint32_t)(start - base);
        }
    }
    const int8_t *const a_base = TA ? args.A + rbase : args.A + (int64_t)row0 * args.lda;
    const int8_t *const b_base = TB ? args.B + (int64_t)col0 * args.ldb : args.B + cbase;
    auto window = [&](int t) {
        const int w = kb + (t < n_full ? t : n_full) * BK;
        return w < K - BK ? w : K - BK;
    };
    // operands of the next stage to request; a short last stage steps to the window that ends at K
    int w_next = window(0);
    const int8_t *pa = a_base + (TA ? (int64_t)w_next * args.lda : (int64_t)w_next);
    const int8_t *pb = b_base + (TB ? (int64_t)w_next : (int64_t)w_next * args.ldb);
    const int w_last = window(n_full);
    auto advance = [&]() {
        const int step = w_last - w_next < BK ? w_last - w_next : BK;
        w_next += step;
        pa += TA ? (int64_t)step * args.lda : (int64_t)step;
        pb += TB ? (int64_t)step : (int64_t)step * args.ldb;
    };
    const uint32_t lds_wave = lds_base + (uint32_t)(g * G_BYTES + wg * 1024);
    // (the branch is inside the asm: the K loop has to stay one basic block)
    auto issue = [&](int t, int slot) {
        const uint32_t dst = lds_wave + (uint32_t)(slot * STAGE_BYTES);
#define CT_LOAD(V, P, O) "s_add_u32 m0, %[d], %[o" #O "]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[v" #V "], %[" #P "]\n\t"
#define CT_BEGIN "s_cmp_lt_i32 %[t], %[n]\n\ts_cbranch_scc0 1f\n\t"
#define CT_IN [d] "s"(dst), [a] "s"(pa), [b] "s"(pb), [t] "s"(t), [n] "s"(n_st), [o0] "n"(0), [o1] "n"(1024 * NW), [o2] "n"(2048 * NW), [o3] "n"(3072 * NW)
        if constexpr (LOADS == 2)
            asm volatile(CT_BEGIN CT_LOAD(0, a, 0) CT_LOAD(1, b, 1) "1:"
                         :: CT_IN, [v0] "v"(voff[0]), [v1] "v"(voff[1]) : "memory", "m0", "scc");
        else if constexpr (LOADS == 3)
            asm volatile(CT_BEGIN CT_LOAD(0, a, 0) CT_LOAD(1, b, 1) CT_LOAD(2, b, 2) "1:"
                         :: CT_IN, [v0] "v"(voff[0]), [v1] "v"(voff[1]), [v2] "v"(voff[LOADS > 2 ? 2 : 0]) : "memory", "m0", "scc");
        else
            asm volatile(CT_BEGIN CT_LOAD(0, a, 0) CT_LOAD(1, a, 1) CT_LOAD(2, b, 2) CT_LOAD(3, b, 3) "1:"
                         :: CT_IN, [v0] "v"(voff[0]), [v1] "v"(voff[1]), [v2] "v"(voff[LOADS > 2 ? 2 : 0]), [v3] "v"(voff[LOADS > 3 ? 3 : 0])
                         : "memory", "m0", "scc");
#undef CT_LOAD
#undef CT_BEGIN
#undef CT_IN
        static_assert((LOADS == 2 && A_LOADS == 1) || (LOADS == 3 && A_LOADS == 1) || (LOADS == 4 && A_LOADS == 2), "the loads above");
        advance();
    };
    // REG: the same pieces through registers (rows at any byte address)
    auto fetch = [&](v4i (&st)[LOADS]) {
#pragma unroll
        for (int q = 0; q < LOADS; ++q)
            if (!RAGGED || q < LOADS - 1 || wg + NW * q < LINES) st[q] = *(const v4i_any *)((q < A_LOADS ? pa : pb) + voff[q]);
        advance();
    };
    // (A's bytes outside the k of the range are zeroed on the way -- a zero adds nothing -- in the last,
    // short stage and in the stages a shorter group only waits through)
    uint32_t minor_mask[4];
    const int tail_off = kb + n_full * BK - window(n_full), tail_end = tail_off + tail;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        minor_mask[d] = 0;
        const int k0 = 16 * ((lane & 3) ^ ((lane >> 4) & 3)) + 4 * d;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k0 + e >= tail_off && k0 + e < tail_end) minor_mask[d] |= 0xffu << (8 * e);
    }
    auto put = [&](int t, int slot, const v4i (&st)[LOADS]) {
        const uint32_t whole = t < n_full ? 0xffffffffu : 0u, part = t <= n_full ? 0xffffffffu : 0u;
#pragma unroll
        for (int q = 0; q < LOADS; ++q) {
            const int line = wg + NW * q;
            if (RAGGED && q == LOADS - 1 && line >= LINES) continue;
            v4i x = st[q];
            if (q >= A_LOADS) {
            } else if constexpr (TA) {
                const int k = (line * 64 + lane) / UA;
                const uint32_t m = (k >= tail_off && k < tail_end ? part : 0u) | whole;
#pragma unroll
                for (int d = 0; d < 4; ++d) x[d] &= (int)m;
            } else {
#pragma unroll
                for (int d = 0; d < 4; ++d) x[d] &= (int)((minor_mask[d] & part) | whole);
            }
            *(v4i *)(ct_smem + slot * STAGE_BYTES + g * G_BYTES + line * 1024 + lane * 16) = x;
        }
    };

    // ---- fragments: four bytes offsets per operand suffice, the rest are immediates ----
    const int tb = lane >> 4, ts = lane & 15;
    const int t_k = 16 * (tb >> 1) + (ts >> 1), t_c = 16 * (tb & 1) + 8 * (ts & 1);
    auto minor_off = [&](int line, int ks) { return line * BK + (((2 * ks + lh) ^ along(line)) * 16); };
    auto major_off = [&](int units, int line0) {     // + k-rows
        const int c = line0 + t_c;
        return t_k * units * 16 + ((c >> 4) ^ swz(units, t_k)) * 16 + (c & 15);
    };
    constexpr int STEPS = BK / 32;                       // k-steps of 32
    int a_off[TA ? MB : STEPS], b_off[TB ? STEPS : NB];
#pragma unroll
    for (int x = 0; x < (TA ? MB : STEPS); ++x)
        a_off[x] = g * G_BYTES + (TA ? major_off(UA, (wr * MB + x) * 32) : minor_off(wr * MB * 32 + li, x));
#pragma unroll
    for (int x = 0; x < (TB ? STEPS : NB); ++x)
        b_off[x] = g * G_BYTES + A_BYTES + (TB ? minor_off(wc * NB * 32 + li, x) : major_off(UB, (wc * NB + x) * 32));
    auto frag_minor = [&](const int8_t *st, int off, int blk) { return *(const v4i *)(st + off + blk * 32 * BK); };
    auto frag_major = [&](const int8_t *st, int units, int off, int ks) {
        const int8_t *p = st + off + ks * 32 * units * 16;
        const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)p);
        const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(p + 8 * units * 16));
        return v4i{lo.x, lo.y, hi.x, hi.y};
    };
    auto read_frags = [&](int slot, int ks, v4i (&a)[MB], v4i (&b)[NB]) {
        const int8_t *st = ct_smem + slot * STAGE_BYTES;
#pragma unroll
        for (int x = 0; x < MB; ++x) a[x] = TA ? frag_major(st, UA, a_off[TA ? x : 0], ks) : frag_minor(st, a_off[TA ? 0 : ks], x);
#pragma unroll
        for (int x = 0; x < NB; ++x) b[x] = TB ? frag_minor(st, b_off[TB ? ks : 0], x) : frag_major(st, UB, b_off[TB ? 0 : x], ks);
    };

    v16i acc[MB][NB];
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[x][y][v] = 0;
    auto mma = [&](const v4i (&a)[MB], const v4i (&b)[NB]) {
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
            for (int y = 0; y < NB; ++y) acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[x], b[y], acc[x][y], 0, 0, 0);
    };
    // the last, short stage: A's bytes outside the k not yet summed are zeroed (a zero adds nothing)
    auto mask_tail = [&](v4i (&a)[MB], int ks) {
        const int off = kb + n_full * BK - window(n_full), end = off + tail;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int k0 = 32 * ks + 16 * lh + 4 * d;
            uint32_t m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k0 + e >= off && k0 + e < end) m |= 0xffu << (8 * e);
#pragma unroll
            for (int x = 0; x < MB; ++x) a[x][d] &= (int)m;
        }
    };

    v4i fa0[MB], fb0[NB], fa1[MB], fb1[NB];
    int t = 0, slot = 0;
    if constexpr (!REG) {
        static_assert(NST >= 3, "a stage is awaited while the next but one is on its way");
#pragma unroll
        for (int d = 0; d < NST - 1; ++d) issue(d, d);
        // stage 0
        if (n_st >= NST - 1) ct_wait_vmcnt<(NST - 2) * LOADS>();
        else ct_wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        auto between = [&](int t, int sl) {     // stage t + 1 has landed, the slot of stage t - 1 takes stage t + NST - 1
            asm volatile("s_cmp_lt_i32 %0, %1\n\t"
                             "s_cbranch_scc1 1f\n\t"
                             "s_waitcnt vmcnt(0)\n"
                             "1:\n\t"
                             "s_waitcnt vmcnt(%2)" :: "s"(t + NST - 2), "s"(n_st), "n"(LOADS * (NST - 3)) : "memory", "scc");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            issue(t + NST - 1, sl == 0 ? NST - 1 : sl - 1);
        };
        if (n_full > 0) {
            read_frags(0, 0, fa0, fb0);
            for (; t < n_full; ++t) {
                const int ns = slot == NST - 1 ? 0 : slot + 1;
                read_frags(slot, 1, fa1, fb1);
                mma(fa0, fb0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (STEPS > 2) {
                    read_frags(slot, 2, fa0, fb0);
                    mma(fa1, fb1);
                    __builtin_amdgcn_sched_barrier(0);
                    read_frags(slot, 3, fa1, fb1);
                    mma(fa0, fb0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                between(t, slot);
                read_frags(ns, 0, fa0, fb0);
                __builtin_amdgcn_sched_barrier(0);
                mma(fa1, fb1);
                slot = ns;
            }
        }
        for (; t < n_st; ++t) {
            if (t == n_full && tail > 0) {
#pragma unroll
                for (int ks = 0; ks < STEPS; ks += 2) {
                    if (STEPS > 2 && 32 * (ks + 2) <= tail_off) continue;      // (summed already)
                    read_frags(slot, ks, fa0, fb0);
                    read_frags(slot, ks + 1, fa1, fb1);
                    mask_tail(fa0, ks);
                    mask_tail(fa1, ks + 1);
                    mma(fa0, fb0);
                    mma(fa1, fb1);
                }
            }
            between(t, slot);
            slot = slot == NST - 1 ? 0 : slot + 1;
        }
    } else {
        // Through registers: two stages on their way in registers, two slots in LDS.
        v4i s0[LOADS], s1[LOADS];
        fetch(s0);
        fetch(s1);
        put(0, 0, s0);
        fetch(s0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        read_frags(0, 0, fa0, fb0);
        // stage u, whose successor is in `nxt`
        auto stage = [&](int u, int sl, v4i (&nxt)[LOADS]) {
            read_frags(sl, 1, fa1, fb1);
            put(u + 1, sl ^ 1, nxt);
            fetch(nxt);
            __builtin_amdgcn_sched_barrier(0);
            mma(fa0, fb0);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            read_frags(sl ^ 1, 0, fa0, fb0);
            __builtin_amdgcn_sched_barrier(0);
            mma(fa1, fb1);
        };
        // (in pairs; a stage past the last has its A zeroed)
        for (; t < n_st; t += 2) {
            stage(t, 0, s1);
            stage(t + 1, 1, s0);
        }
    }

    // ---- where a place of the tile lies in R ----
    // (rows and columns counted from the tile's base, so that an output is a 32-bit offset from one
    // wave-uniform address)
    auto row_of = [&](int p, bool &own) {
        if (TA) {
            const int u = row0 + (p & ~15);
            const int row = (u < M - 16 ? u : M - 16) + (p & 15);
            own = row >= u;
            return row - rbase;
        }
        own = row0 + p < M;
        return p;
    };
    auto col_of = [&](int p, bool &own) {
        if (!TB) {
            const int u = col0 + (p & ~15);
            const int col = (u < N - 16 ? u : N - 16) + (p & 15);
            own = col >= u;
            return col - cbase;
        }
        own = col0 + p < N;
        return p;
    };
    int32_t *const r_base = args.R + (int64_t)rbase * args.ldr + cbase;

    // ---- write-back: parts of 64 or 32 rows through an LDS image (the ring is free now) ----
    // The first group's waves store their accumulators (element v of lane l is R[8*(v/4) + 4*(l/32) +
    // v%4][l%32] of its 32 x 32 block), the other groups add theirs, and all waves carry the image to R
    // in 16-byte pieces of rows.  Every other group of four image rows has its 128-byte halves exchanged, so
    // that the two half-waves of a scatter, four rows apart, use different banks.
    constexpr int NWT = WR * WC * WK, PR = BN / (4 * NWT) > 4 ? 32 : 64;   // (four pieces of R in a lane's registers: more spill)
    constexpr int NA = (PR * BN + 256 * NWT - 1) / (256 * NWT), ROW_U = BN / 4;
    static_assert(!KS || PR * BN % (256 * NWT) == 0, "the image's pieces divide over the waves");
    int32_t *const img = (int32_t *)ct_smem;
    auto img_at = [](int r, int c) { return r * BN + (BN > 32 ? c ^ (((r >> 2) & 1) << 5) : c); };
    auto scatter = [&](int part, auto add) {
#pragma unroll
        for (int x = 0; x < MB; ++x) {
            if ((wr * MB + x) * 32 / PR != part) continue;
#pragma unroll
            for (int y = 0; y < NB; ++y)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = (wr * MB + x) * 32 % PR + 8 * (v >> 2) + 4 * lh + (v & 3);
                    int32_t *const dst = img + img_at(r, (wc * NB + y) * 32 + li);
                    if (decltype(add)::value) atomicAdd(dst, acc[x][y][v]);
                    else *dst = acc[x][y][v];
                }
        }
    };
    auto image = [&](int part) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // the ring, or the part before, is no longer read
        if (g == 0) scatter(part, std::false_type());
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if constexpr (WK > 1) {
            if (g > 0) scatter(part, std::true_type());
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    };
    if (KS) {
        // Several workgroups own this tile.  64 neighbours of a row per instruction: a wave's atomic adds to 256
        // contiguous bytes go four times as fast as to every fourth value of 1024 (0.43 against 0.11 T adds/s).
#pragma unroll
        for (int part = 0; part < BM / PR; ++part) {
            image(part);
#pragma unroll
            for (int i = 0; i < 4 * NA; ++i) {
                const int idx = i * (64 * NWT) + tid, r = idx / BN, c = idx % BN;
                bool orow, ocol;
                const int row = row_of(part * PR + r, orow), col = col_of(c, ocol);
                if (orow && ocol) atomicAdd(r_base + (uint32_t)row * (uint32_t)args.ldr + (uint32_t)col, img[img_at(r, c)]);
            }
        }
        return;
    }
#pragma unroll
    for (int part = 0; part < BM / PR; ++part) {
        uint32_t off[NA];
        bool all[NA];
        v4i old[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int idx = i * (64 * NWT) + tid, r = idx / ROW_U, c = idx % ROW_U * 4;
            bool orow, o0, o3;
            const int row = row_of(part * PR + r, orow), col = col_of(c, o0);
            if (PR * BN % (256 * NWT) != 0) orow = orow && r < PR;
            (void)col_of(c + 3, o3);
            off[i] = (uint32_t)row * (uint32_t)args.ldr + (uint32_t)col;
            all[i] = orow && o0 && o3;
            old[i] = v4i{0, 0, 0, 0};
            if (all[i] && !args.assign) old[i] = NT ? __builtin_nontemporal_load((const v4i_r *)(r_base + off[i])) : *(const v4i_r *)(r_base + off[i]);
        }
        // (edges after the whole pieces, so that only waves that have one wait between loads of one register)
        if (!args.assign) {
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int idx = i * (64 * NWT) + tid, r = idx / ROW_U, c = idx % ROW_U * 4;
                bool orow;
                (void)row_of(part * PR + r, orow);
                if (PR * BN % (256 * NWT) != 0) orow = orow && r < PR;
                if (orow && !all[i]) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bool o;
                        (void)col_of(c + e, o);
                        if (o) old[i][e] = r_base[off[i] + e];
                    }
                }
            }
        }
        image(part);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int idx = i * (64 * NWT) + tid, r = idx / ROW_U, c = idx % ROW_U * 4;
            v4i sum = *(const v4i *)(img + img_at(r, c));
            if (all[i]) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = (int)((uint32_t)sum[e] + (uint32_t)old[i][e]);
                if (NT) __builtin_nontemporal_store(sum, (v4i_r *)(r_base + off[i]));
                else *(v4i_r *)(r_base + off[i]) = sum;
                continue;
            }
            bool orow;
            (void)row_of(part * PR + r, orow);
            if (PR * BN % (256 * NWT) != 0) orow = orow && r < PR;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool o;
                (void)col_of(c + e, o);
                if (!(o && orow)) continue;
                r_base[off[i] + e] = (int)((uint32_t)sum[e] + (uint32_t)old[i][e]);
            }
        }
    }
}

template <int MB, int NB, int WR, int WC, int WK, int NST, bool TA, bool TB, bool REG, bool KS, bool NT = false, int BK = CT_BK>
static hipError_t launch_tile(int parts, const CountTileArgs &args, hipStream_t s)
{
    constexpr int BM = 32 * MB * WR, BN = 32 * NB * WC, RING = (REG ? 2 : NST) * WK * BK * (BM + BN), IMAGE = 64 * BN * 4;
    constexpr int LDS = RING > IMAGE ? RING : IMAGE;
    auto *const kernel = &count_i8_tile_kernel<MB, NB, WR, WC, WK, NST, TA, TB, REG, KS, NT, BK>;
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (granted != hipSuccess) return granted;
    const int64_t grid = xcd_grid((args.M + BM - 1) / BM, (args.N + BN - 1) / BN);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    CountTileArgs a = args;
    return launch_row_of_blocks(a, grid, 64 * WR * WC * WK, [&](unsigned n) {
        hipLaunchKernelGGL(kernel, dim3(n, (unsigned)parts), dim3(64 * WR * WC * WK), LDS, s, a);
    });
}

template <bool TA, bool TB, bool REG>
static hipError_t launch_tile_plan(const CountTilePlan &plan, const CountTileArgs &a, hipStream_t s)
{
    switch (plan.tile) {
    case CT_256:
        if (a.bypass) return launch_tile<2, 2, 4, 4, 1, 4, TA, TB, REG, false, true>(1, a, s);
        return launch_tile<2, 2, 4, 4, 1, 4, TA, TB, REG, false>(1, a, s);
    case CT_128x256:
        if constexpr (!REG) {
            if (plan.alone) return launch_tile<2, 2, 2, 4, 1, 6, TA, TB, REG, false>(1, a, s);
            if (a.bypass) return launch_tile<2, 2, 2, 4, 1, 3, TA, TB, REG, false, true>(1, a, s);
            return launch_tile<2, 2, 2, 4, 1, 3, TA, TB, REG, false>(1, a, s);
        }
        return hipErrorInvalidValue;
    case CT_192x256:      // (a transposed A's k-rows have 12 units there, which the exchange of units does not fit)
        if constexpr (REG && !TA) return launch_tile<2, 2, 3, 4, 1, 4, TA, TB, REG, false>(1, a, s);
        return hipErrorInvalidValue;
    case CT_128:
        if constexpr (!REG) {
            if (plan.deep && plan.parts > 1) return launch_tile<2, 1, 2, 4, 1, 4, TA, TB, REG, true, false, 128>(plan.parts, a, s);
            if (plan.deep) return launch_tile<2, 1, 2, 4, 1, 4, TA, TB, REG, false, false, 128>(1, a, s);
        }
        if (plan.parts > 1) return launch_tile<2, 1, 2, 4, 1, 4, TA, TB, REG, true>(plan.parts, a, s);
        return launch_tile<2, 1, 2, 4, 1, 4, TA, TB, REG, false>(1, a, s);
    default:
        if constexpr (!REG && !(TA && !TB)) {
            if (plan.deep && plan.parts > 1) return launch_tile<1, 1, 2, 2, 2, 4, TA, TB, REG, true, false, 128>(plan.parts, a, s);
            if (plan.deep) return launch_tile<1, 1, 2, 2, 2, 4, TA, TB, REG, false, false, 128>(1, a, s);
        }
        if (plan.parts > 1) return launch_tile<1, 1, 2, 2, 2, 4, TA, TB, REG, true>(plan.parts, a, s);
        return launch_tile<1, 1, 2, 2, 2, 4, TA, TB, REG, false>(1, a, s);
    }
}

hipError_t launch_count_i8_tile(int trans, const CountTilePlan &plan, const CountTileArgs &args, hipStream_t s)
{
    CountTileArgs a = args;
    a.kpart = plan.kpart;
    a.kgroup = plan.kgroup;
    a.block_base = 0;
    switch (trans + (plan.through_registers ? 4 : 0)) {
    case 0: return launch_tile_plan<false, false, false>(plan, a, s);
    case 1: return launch_tile_plan<true, false, false>(plan, a, s);
    case 2: return launch_tile_plan<false, true, false>(plan, a, s);
    case 3: return launch_tile_plan<true, true, false>(plan, a, s);
    case 4: return launch_tile_plan<false, false, true>(plan, a, s);
    case 5: return launch_tile_plan<true, false, true>(plan, a, s);
    case 6: return launch_tile_plan<false, true, true>(plan, a, s);
    default: return launch_tile_plan<true, true, true>(plan, a, s);
    }
}

}  // namespace amulet
