// Tile kernels of the predicate tasks, fp32 and fp64: 32 x 64 or 16 x 64 outputs per workgroup of eight
// waves that share the tile's K.  The built-in choice for problems that give the wide tiles of
// mmlike_valu_impl.h (16 or 32 rows x 256 columns, one wave per 4 rows, K whole) too few waves to fill
// the chip, or columns to waste; in fp64 at nearly every size.  (Which one a call gets, and with
// which split of K: tile_wanted, choose_tile_plan.)
//
// What bounded such problems: a wave of the wide kernels owns 4 x 256 outputs over all of its K,
// so 512^3 is 256 waves for 1024 SIMDs, and a wave alone on its SIMD issues one vector instruction
// in four clocks where two or more issue two; splitting K further over workgroups pays an atomic
// add per output and part.  A column count just over a multiple of 256 fills a quarter of a tile.
//
// Here
//   * a wave owns 16 x 64 outputs, a lane 4 x 4 of them (4 groups of 16 lanes, one group per 4 rows): A and
//     B both come from LDS as 16-byte units, two reads per 16 products in fp32;
//   * the tile's K is cut into 4 or 8 ranges, one per group of waves; their sums meet in LDS at the end,
//     in a fixed order, and every wave finishes a part of the tile: no atomics, and the same bits
//     every time, until K is also split over workgroups (TilePlan::parts);
//   * operands stream HBM -> LDS (global_load_lds_dwordx4) through a ring of NST stages of 64 bytes of k,
//     each group its own, one barrier per stage.  A lane may fetch from any element address, so any
//     size, pitch and layout runs the same loop: a row or column past the edge is replaced by the last
//     one inside, a unit of rows (columns) that would end past the edge by the one that ends AT it -- the
//     lane then owns those rows (columns) and leaves the ones its neighbour owns alone -- and the last,
//     short stage of a k range by the window that ends at K, of which only the k not yet summed are used;
//   * a stage's barrier sits one k into its last chunk of V k: by then a wave holds all of the stage's
//     fragments, and those of the next stage are read while the rest of the chunk computes.
//
// Bound: vector-ALU issue (fp32 9.1-9.2 clocks per 64 products of discount and boost in a register-only
// loop, 6.6 count; fp64 16 of an ideal 16), and below about 1024^3 the launch, the first loads and the
// write-back, 5 us in all.  LDS reads are 40-60 % of what a compute unit can do.  Measured, wide / tile, us:
// fp32 discount 64^3 12.9 / 5.0, 256^3 13.5 / 5.4, 512^3 31.8 / 13.2, 1024^3 80 / 72, 1536^3 245 / 228; fp64
// discount 256^3 16.3 / 7.5, 512^3 40.5 / 22.8, 4096^3 8155 / 7823 (17.6 TFLOP/s), count 6146 / 5650.  From 2048^3 on
// the wide fp32 kernel is as fast or faster (33.8 against 32.5 TFLOP/s at 4096^2): half the LDS reads.
//
// FAST: the count by rounding (count_rounding.h), thresholds that face rows, columns or all: the factor is multiplied to four operands
// of each k after they are read.  us, by comparison / so: 768^3 31.7 / 28.2, 1003 x 1501 x 777 66.3 / 58.2, 3262 x 288 x 5014 262 / 225, 640^3 20.7 /
// 19.8, 128 x 4096 x 512 17.5 / 16.8, but 2048 x 300 x 200 14.6 / 14.8, 256^3 5.0 / 5.4: looking at the thresholds and the waves' words at the end take
// 0.4 us, so from 15 us of plan on.  Thresholds of zero have a loop of their own (a factor on both operands, none to look at): 768^3
// 32.8 / 29.1, 1003 x 1501 x 777 68.0 / 60.9, 1536^3 facing rows 197 / 170.
//
// LDS layout of a group's stage: A, then B.  An operand whose lines run along k (row-major A, transposed B)
// is kept as lines of 4 units, the other kind as k-rows of units.  16 lanes are served per clock: of A they
// read one unit (broadcast), of row-major B 16 neighbouring units; transposed B takes columns lc, lc + 16, ...
// to a lane and keeps unit u of column c at u ^ ((c >> 2) & 3), so that 16 lanes read 16 distinct bank groups.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "amulet_internal.h"
#include "count_rounding.h"

#ifndef AMULET_MMLIKE_TILE_IMPL_H
#define AMULET_MMLIKE_TILE_IMPL_H

// the LDS-DMA asm below sets M0 itself and says so in its clobber list
#pragma clang diagnostic ignored "-Winline-asm"

namespace amulet {

typedef __attribute__((address_space(3))) void *tile_lds_ptr;
extern __shared__ __attribute__((aligned(16))) char tile_smem[];

enum { BY_COMPARISON = 0, BY_ROUNDING = 1, BY_ROUNDING_ZERO = 2 };     // how the count decides its predicate

template <typename T> struct TileVec;
template <> struct TileVec<float> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct TileVec<double> { typedef double type __attribute__((ext_vector_type(2))); };

template <typename T, int TASK> struct TileAcc { typedef T type; };
template <typename T> struct TileAcc<T, TASK_COUNT_GT> { typedef int type; };

template <int N> __device__ __forceinline__ void tile_wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Resident waves per SIMD the registers are held to: two workgroups to a compute unit, but with 32 registers
// of thresholds (thres[i][j] in fp64) one: held to four waves that form spills inside the K loop (up to 26 scratch
// accesses per 8 k), every other form fits its 128.
template <typename T, int TF> constexpr int tile_waves() { return sizeof(T) == 8 && TF == THRES_ELEM ? 2 : 4; }

// LDS of a workgroup: the ring, and behind the image its sums meet in a word of each wave's
constexpr int tile_ring(int wm, int wn, int wk, int nst) { return nst * wk * (1024 * wm + 4096 * wn); }
constexpr int tile_sums(int sz, int wm, int wn, int wk) { return wm * wn * wk * 1024 * sz; }

template <typename T, int TASK, int TF, int TRANS, int WM, int WN, int WK, int NST, bool FAST>
__global__ void __launch_bounds__(64 * WM * WN * WK) __attribute__((amdgpu_waves_per_eu(tile_waves<T, TF>(), tile_waves<T, TF>())))
mmlike_tile_kernel(const TileArgs<T> args)
{
    typedef typename TileVec<T>::type vec;
    typedef typename TileAcc<T, TASK>::type acc_t;
    constexpr int SZ = sizeof(T), V = 16 / SZ, BK = 4 * V;      // elements of a 16-byte unit; k of a stage
    constexpr int TR = 16 * WM, TC = 64 * WN;                   // rows and columns of the tile
    constexpr int A_BYTES = 1024 * WM, G_BYTES = A_BYTES + 4096 * WN, STAGE_BYTES = WK * G_BYTES;
    constexpr int NW = WM * WN, LINES = WM + 4 * WN, LOADS = (LINES + NW - 1) / NW;
    constexpr int H = 4 / V;                                    // units in four elements
    constexpr bool TA = (TRANS & 1) != 0, TB = (TRANS & 2) != 0;

    const int M = args.M, N = args.N, K = args.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = wave / NW, wg = wave % NW, wm = wg / WN, wn = wg % WN;
    const int lr = lane >> 4, lc = lane & 15;

    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, (M + TR - 1) / TR, (N + TC - 1) / TC, tm, tn)) return;
    const int row0 = __builtin_amdgcn_readfirstlane(tm * TR), col0 = __builtin_amdgcn_readfirstlane(tn * TC);

    const bool ksplit = gridDim.y > 1;
    const int part0 = (int)blockIdx.y * args.kpart;
    const int part_len = K - part0 < args.kpart ? K - part0 : args.kpart;
    const int kb = part0 + g * args.kgroup;
    int klen = part_len - g * args.kgroup;
    klen = klen < 0 ? 0 : klen < args.kgroup ? klen : args.kgroup;
    const int n_full = klen / BK, tail = klen - n_full * BK;
    const int n_st = ((args.kgroup < part_len ? args.kgroup : part_len) + BK - 1) / BK;

    // ---- operand stream: which 16 bytes each lane fetches, LOADS wave-loads of 1 KB per wave and stage ----
    // A wave-uniform base (the tile's origin, moved back where the first unit ends at the edge, and
    // the stage's k) plus a 32-bit offset per lane that never changes.  (Where the lines do not divide
    // evenly over the group's waves some are fetched twice, so that every wave waits for the same count.)
    uint32_t voff[LOADS], ldst[LOADS];
    bool is_a[LOADS];
    const int rbase = TA && row0 > M - V ? M - V : row0, cbase = !TB && col0 > N - V ? N - V : col0;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(tile_lds_ptr)tile_smem;
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
        int line = wg + NW * q;
        if (LINES % NW != 0 && line >= LINES) line -= LINES;
        is_a[q] = line < WM;
        ldst[q] = lds_base + (uint32_t)(g * G_BYTES + line * 1024);
        if (is_a[q]) {
            const int s = line * 64 + lane;
            if (TA) {
                const int k = s / (TR / V), u = s % (TR / V);
                const int start = row0 + u * V < M - V ? row0 + u * V : M - V;
                voff[q] = ((uint32_t)k * (uint32_t)args.lda + (uint32_t)(start - rbase)) * (uint32_t)SZ;
            } else {
                const int r = row0 + (s >> 2) < M ? s >> 2 : M - 1 - row0;
                voff[q] = ((uint32_t)r * (uint32_t)args.lda + (uint32_t)((s & 3) * V)) * (uint32_t)SZ;
            }
        } else {
            const int s = (line - WM) * 64 + lane;
            if (TB) {
                const int c = s >> 2, u = (s & 3) ^ ((c >> 2) & 3);
                const int cc = col0 + c < N ? c : N - 1 - col0;
                voff[q] = ((uint32_t)cc * (uint32_t)args.ldb + (uint32_t)(u * V)) * (uint32_t)SZ;
            } else {
                const int k = s / (TC / V), u = s % (TC / V);
                const int start = col0 + u * V < N - V ? col0 + u * V : N - V;
                voff[q] = ((uint32_t)k * (uint32_t)args.ldb + (uint32_t)(start - cbase)) * (uint32_t)SZ;
            }
        }
    }
    const T *const a_base = TA ? args.A + rbase : args.A + (int64_t)row0 * args.lda;
    const T *const b_base = TB ? args.B + (int64_t)col0 * args.ldb : args.B + cbase;
    // first k of stage t's window; the windows of stages past the range are loaded and not used
    auto window = [&](int t) {
        const int w = kb + (t < n_full ? t : n_full) * BK;
        return w < K - BK ? w : K - BK;
    };
    // (the branch is inside the asm: the K loop's arithmetic has to stay one basic block, see below)
    auto issue = [&](int t, int slot) {
        const int w = window(t);
        const T *const pa = a_base + (TA ? (int64_t)w * args.lda : (int64_t)w);
        const T *const pb = b_base + (TB ? (int64_t)w : (int64_t)w * args.ldb);
#pragma unroll
        for (int q = 0; q < LOADS; ++q) {
            const T *const p = is_a[q] ? pa : pb;
            asm volatile("s_cmp_lt_i32 %3, %4\n\t"
                         "s_cbranch_scc0 1f\n\t"
                         "s_mov_b32 m0, %2\n\t"
                         "s_nop 0\n\t"
                         "global_load_lds_dwordx4 %0, %1\n"
                         "1:"
                         :
                         : "v"(voff[q]), "s"(p), "s"(ldst[q] + (uint32_t)(slot * STAGE_BYTES)), "s"(t), "s"(n_st)
                         : "memory", "m0", "scc");
        }
    };
#pragma unroll
    for (int d = 0; d < NST; ++d) issue(d, d);

    // ---- row and column of R at a place of the wave's 16 x 64, and whether it is written from here ----
    auto row_at = [&](int p, bool &own) {
        if (TA) {
            const int u = row0 + wm * 16 + p / V * V;
            const int row = (u < M - V ? u : M - V) + p % V;
            own = row >= u;
            return row;
        }
        const int row = row0 + wm * 16 + p;
        own = row < M;
        return own ? row : M - 1;
    };
    auto col_at = [&](int p, bool &own) {
        if (TB) {
            const int col = col0 + wn * 64 + p;
            own = col < N;
            return own ? col : N - 1;
        }
        const int u = col0 + wn * 64 + p / V * V;
        const int col = (u < N - V ? u : N - V) + p % V;
        own = col >= u;
        return col;
    };
    // (of lane l's products)
    auto row_of = [&](int l, int r, bool &own) { return row_at((l >> 4) * 4 + r, own); };
    auto col_of = [&](int l, int c, bool &own) { return col_at(TB ? (l & 15) + 16 * c : c / V * (16 * V) + (l & 15) * V + c % V, own); };

    static_assert(!FAST || (SZ == 4 && TASK == TASK_COUNT_GT && TF != THRES_ELEM), "the count by rounding");
    static_assert(!FAST || tile_sums(SZ, WM, WN, WK) + 64 <= tile_ring(WM, WN, WK, NST), "the waves' words");
    // Thresholds and factors in registers for the whole K loop.  (The count reads its predicate from
    // the sign of th - p, which takes a threshold of -0 for a negative number: held as th + 0.)
    auto held = [](T t) { return TASK == TASK_COUNT_GT ? t + (T)0 : t; };
    T th[TF == THRES_ELEM || TF == THRES_ROW ? 4 : 1][TF == THRES_ELEM || TF == THRES_COL ? 4 : 1];
    T q[4];
    bool own_dummy;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int col = col_of(lane, c, own_dummy);
        q[c] = (T)1;
        if constexpr (TASK == TASK_DISCOUNT) q[c] = (T)1 - args.dis[col];
        if constexpr (TF == THRES_COL) th[0][c] = held(args.thres[col]);
        if constexpr (TF == THRES_ELEM) {
#pragma unroll
            for (int r = 0; r < 4; ++r) th[r][c] = held(args.thres[(int64_t)row_of(lane, r, own_dummy) * args.ldt + col]);
        }
    }
    if constexpr (TF == THRES_ROW) {
#pragma unroll
        for (int r = 0; r < 4; ++r) th[r][0] = held(args.thres[row_of(lane, r, own_dummy)]);
    }
    if constexpr (TF == THRES_CONST) {
        th[0][0] = held(args.thres[0]);
        asm volatile("" : "+v"(th[0][0]));
    }
    auto thr = [&](int r, int c) { return th[TF == THRES_ELEM || TF == THRES_ROW ? r : 0][TF == THRES_ELEM || TF == THRES_COL ? c : 0]; };

    // partial sums over 64 k and main accumulators (fp32), one level (fp64), or predicate bits of 32 k
    // and their count
    acc_t part[4][4], mainacc[4][4];
    uint32_t bits[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) { part[r][c] = 0; mainacc[r][c] = 0; bits[r][c] = 0; }
    // FAST, the count by rounding (count_rounding.h): sums, factors and rounding constants of the thresholds, the largest operand
    // with its factor
    constexpr int NS = TF == THRES_ROW || TF == THRES_COL ? 4 : 1;
    T sum[4][4], gain[NS], sway[NS], most = 0;
    bool quick = false, zero = false;
    if constexpr (FAST) {
        bool every = args.kgroup <= COUNT_ROUNDING_K, none = every;
        T neg[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const T t = thr(TF == THRES_ROW ? i : 0, i);
            every = count_rounding(t, gain[i], sway[i], neg[i]) && every;
            none = t == 0 && none;
        }
        quick = __builtin_amdgcn_ballot_w64(!every) == 0;
        zero = __builtin_amdgcn_ballot_w64(!none) == 0;
        if (quick)
#pragma unroll
            for (int i = 0; i < NS; ++i) th[TF == THRES_ROW ? i : 0][TF == THRES_COL ? i : 0] = neg[i];
        if constexpr (TF == THRES_CONST) asm volatile("" : "+v"(gain[0]), "+v"(sway[0]), "+v"(th[0][0]));
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[r][c] = COUNT_ROUNDING_ZERO;
    }
    // one k of the lane's 4 x 4: the factors go on the operand that faces the thresholds; a threshold of zero's on both, where
    // an overflow is always as good as the value (count_rounding.h)
    auto fast_k = [&](const T (&a)[4], const T (&b)[4], auto fast) {
        if constexpr (FAST) {
            constexpr bool ROW = TF == THRES_ROW;
            if constexpr (decltype(fast)::value == BY_ROUNDING_ZERO) {
                T x[4], y[4], neg[4], s[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[i] = a[i] * COUNT_ZERO_A; y[i] = b[i] * COUNT_ZERO_B; neg[i] = COUNT_ZERO_NEG; s[i] = 1; }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    count_by_rounding4(x[r], y, neg, s, sum[r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                T x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = (ROW ? a[i] : b[i]) * gain[i % NS];
                most = __builtin_fmaxf(most, __builtin_fmaxf(__builtin_fabsf(x[0]), __builtin_fabsf(x[1])));
                most = __builtin_fmaxf(most, __builtin_fmaxf(__builtin_fabsf(x[2]), __builtin_fabsf(x[3])));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    T neg[4], s[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) { neg[c] = thr(r, c); s[c] = sway[ROW ? r : c % NS]; }
                    count_by_rounding4(ROW ? x[r] : a[r], ROW ? b : x, neg, s, sum[r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };

    auto product = [&](T a, T b, int r, int c) {     // one product on its own (the K remainder)
        const T t = thr(r, c);
        if constexpr (TASK == TASK_DISCOUNT) {
            const T p = a * b;
            part[r][c] = __builtin_elementwise_fma(p, p > t ? q[c] : (T)1, part[r][c]);
        } else if constexpr (TASK == TASK_BOOST) {
            part[r][c] = __builtin_elementwise_fma(a, b, part[r][c]);
            part[r][c] += __builtin_elementwise_max(__builtin_elementwise_fma(a, b, -t), (T)0);
        } else {
            const T p = a * b;
            part[r][c] += (int)(p > t);
        }
    };

    // One chunk of V k, four units of each operand; side(kk) after the products of k kk, where the units
    // whose last use that was may be refilled.  Per product: discount fp32 multiply, compare, select,
    // fma as one software pipeline (compare i, multiply i + 1, fma i - 1, select i: see mmlike_valu_impl.h);
    // discount fp64 under the execution mask; boost p + max(p - th, 0) with the unrounded product inside its two fused
    // operations, one product at a time (multiply, fma, max, add on the rounded one, max(p, 2p - th), is no
    // faster: us, that / this, 1024^3 70.3 / 70.8, 1003 x 1501 x 777 81.9 / 82.2, fp64 2048^3 978 / 968; in groups of
    // four 71.6, 82.5, 962); count multiply, subtract, and the sign bit shifted into a register of 32 (in fp64 the
    // sign bit of the high half: 20.7 -> 23.7 TFLOP/s at 2048^3 against compare, select, add).
    auto a_of = [](const vec (&v)[4], int r, int kk) -> T { return TA ? v[kk * H + r / V][r % V] : v[r][kk]; };
    auto b_of = [](const vec (&v)[4], int kk, int c) -> T { return TB ? v[c][kk] : v[kk * H + c / V][c % V]; };
    auto chunk = [&](const vec (&a)[4], const vec (&b)[4], auto side, auto fast) {
        if constexpr (decltype(fast)::value) {
#pragma unroll
            for (int kk = 0; kk < V; ++kk) {
                T ak[4], bk[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { ak[i] = a_of(a, i, kk); bk[i] = b_of(b, kk, i); }
                fast_k(ak, bk, fast);
                side(kk);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if constexpr (TASK == TASK_DISCOUNT && sizeof(T) == 8) {
            const uint64_t active = __builtin_amdgcn_read_exec();
#pragma unroll
            for (int kk = 0; kk < V; ++kk) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    T p[4][2];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < 2; ++c) p[r][c] = a_of(a, r, kk) * b_of(b, kk, 2 * h + c);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < 2; ++c)
                            asm volatile("v_cmpx_gt_f64_e32 vcc, %0, %1\n\tv_mul_f64 %0, %0, %2\n\ts_mov_b64 exec, %3"
                                         : "+v"(p[r][c])
                                         : "v"(thr(r, 2 * h + c)), "v"(q[2 * h + c]), "s"(active)
                                         : "vcc");
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < 2; ++c) part[r][2 * h + c] += p[r][c];
                }
                side(kk);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if constexpr (TASK == TASK_DISCOUNT) {
            constexpr int NP = V * 16;
            T p[NP + 1], sel[NP];
            p[0] = a_of(a, 0, 0) * b_of(b, 0, 0);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int r = (i / 4) % 4, c = i % 4;
                const bool m = p[i] > thr(r, c);
                __builtin_amdgcn_sched_barrier(0);
                if (i + 1 < NP) p[i + 1] = a_of(a, ((i + 1) / 4) % 4, (i + 1) / 16) * b_of(b, (i + 1) / 16, (i + 1) % 4);
                __builtin_amdgcn_sched_barrier(0);
                if (i > 0) part[((i - 1) / 4) % 4][(i - 1) % 4] = __builtin_elementwise_fma(p[i - 1], sel[i - 1], part[((i - 1) / 4) % 4][(i - 1) % 4]);
                __builtin_amdgcn_sched_barrier(0);
                sel[i] = m ? q[c] : (T)1;
                __builtin_amdgcn_sched_barrier(0);
                // (the last k's products are begun before the one of the next k reads its operands)
                if (i % 16 == 15) side(i / 16);
                __builtin_amdgcn_sched_barrier(0);
            }
            part[3][3] = __builtin_elementwise_fma(p[NP - 1], sel[NP - 1], part[3][3]);
        } else {
#pragma unroll
            for (int kk = 0; kk < V; ++kk) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (TASK == TASK_BOOST) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const T d = __builtin_elementwise_fma(a_of(a, r, kk), b_of(b, kk, c), -thr(r, c));
                            part[r][c] = __builtin_elementwise_fma(a_of(a, r, kk), b_of(b, kk, c), part[r][c]);
                            part[r][c] += __builtin_elementwise_max(d, (T)0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        T p[4], d[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) p[c] = a_of(a, r, kk) * b_of(b, kk, c);
#pragma unroll
                        for (int c = 0; c < 4; ++c) d[c] = thr(r, c) - p[c];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t hi = sizeof(T) == 4 ? __builtin_bit_cast(uint32_t, (float)d[c]) : (uint32_t)(__builtin_bit_cast(uint64_t, (double)d[c]) >> 32);
                            bits[r][c] = __builtin_amdgcn_alignbit(bits[r][c], hi, 31);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                side(kk);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    constexpr int FLUSH_STAGES = (TASK == TASK_COUNT_GT ? 32 : 64) / BK;
    auto flush = [&](auto fast) {
        if (decltype(fast)::value) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if constexpr (TASK == TASK_COUNT_GT) {
                    part[r][c] += __builtin_popcount(bits[r][c]);
                    bits[r][c] = 0;
                } else if constexpr (sizeof(T) == 4) {
                    mainacc[r][c] += part[r][c];
                    part[r][c] = 0;
                }
            }
    };

    // ---- fragment reads ----
    const int a_lds = g * G_BYTES + (TA ? ((wm * 16 + lr * 4) / V) * 16 : (wm * 16 + lr * 4) * 64);
    const int b_lds = g * G_BYTES + A_BYTES + (TB ? (wn * 64 + lc) * 64 : (wn * (64 / V) + lc) * 16);
    const int b_swz = TB ? ((lc >> 2) & 3) : 0;
    auto read_a = [&](const char *st, int c, int i) {
        return *(const vec *)(st + a_lds + (TA ? (c * V + i / H) * (TR * SZ) + (i % H) * 16 : i * 64 + c * 16));
    };
    auto read_b = [&](const char *st, int c, int i) {
        return *(const vec *)(st + b_lds + (TB ? i * 1024 + (c ^ b_swz) * 16 : (c * V + i / H) * (TC * SZ) + (i % H) * 256));
    };
    // units that run across k are free after their k and refilled in place; units that run along k all stay
    // in use to the chunk's end and have a second set
    constexpr int AS = TA ? 1 : 2, BS = TB ? 2 : 1;     // register sets

    // until stage t has landed: the loads of stages t + 1 ... t + NST - 2 may still be on their way
    auto wait_for = [&](int t, int later) {
        if (later == 0) { tile_wait_vmcnt<0>(); return; }
        asm volatile("s_cmp_lt_i32 %0, %1\n\t"
                     "s_cbranch_scc1 1f\n\t"
                     "s_waitcnt vmcnt(0)\n"
                     "1:\n\t"
                     "s_waitcnt vmcnt(%2)" :: "s"(t + later), "s"(n_st), "n"(LOADS * (NST - 2)) : "memory", "scc");
    };
    // the end of stage t: every wave holds its last fragments, stage t + 1 has landed, the slot of
    // stage t takes the request for stage t + NST
    auto next_stage = [&](int t, int sl) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_for(t + 1, NST - 2);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(t + NST, sl);
    };
    if constexpr (FAST) {
        auto k_loop = [&](auto fast) {
#include "mmlike_tile_k_loop.inc"
        };
        auto counted = [&]() {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) part[r][c] = (int)(sum[r][c] - COUNT_ROUNDING_ZERO);
        };
        if (quick) {
            k_loop(std::integral_constant<int, BY_ROUNDING>());
            counted();
        } else if (zero) {
            k_loop(std::integral_constant<int, BY_ROUNDING_ZERO>());
            counted();
        } else {
            k_loop(std::integral_constant<int, BY_COMPARISON>());
        }
        // an operand left fp32 with its factor, in some wave: all of the tile again, by comparison.  (The ring is free but for what
        // waves still read ahead and never use.)
        int *const redo = (int *)(tile_smem + tile_ring(WM, WN, WK, NST) - 64);
        const bool out = quick && __builtin_amdgcn_ballot_w64(most == __builtin_inff()) != 0;
        if (lane == 0) redo[wave] = out ? 1 : 0;
        __syncthreads();
        if (__builtin_amdgcn_ballot_w64(redo[lane & 7] != 0) != 0) {
#pragma unroll
            for (int i = 0; i < NS; ++i)
                th[TF == THRES_ROW ? i : 0][TF == THRES_COL ? i : 0] =
                    held(args.thres[TF == THRES_ROW ? row_of(lane, i, own_dummy) : TF == THRES_COL ? col_of(lane, i, own_dummy) : 0]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) part[r][c] = 0;
            __syncthreads();
#pragma unroll
            for (int d = 0; d < NST; ++d) issue(d, d);
            k_loop(std::integral_constant<int, BY_COMPARISON>());
        }
    } else {
        constexpr std::integral_constant<int, BY_COMPARISON> fast;
#include "mmlike_tile_k_loop.inc"
    }
    auto result = [&](int r, int c) -> acc_t { return TASK == TASK_COUNT_GT || sizeof(T) == 8 ? part[r][c] : mainacc[r][c]; };

    // ---- sum over the k groups through LDS, write-back ----
    constexpr int VALS = 16 / WK;          // values of the micro-tile this wave finishes
    constexpr int U = VALS < V ? VALS : V; // of which U at a time are neighbours in a row of R (row-major B)
    acc_t out[VALS];
    const int v0 = g * VALS;
    __syncthreads();
    // (opaque from here on, or the rows and columns of the write-back are computed with those of the thresholds, before
    // the K loop, and held through it: up to 11 registers more than the 128 there are)
    int l = lane;
    asm volatile("" : "+v"(l));
    acc_t *const img = (acc_t *)tile_smem;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) img[(((g * NW + wg) * 4 + r) * 64 + l) * 4 + c] = result(r, c);
    __syncthreads();
    if (ksplit) {
        // Several workgroups own this tile: hardware float adds, in whatever order, 64 neighbours of a row
        // at a time.  A wave's atomic adds to 256 contiguous bytes go four times as fast as to every fourth
        // value of 1024: fp32 0.084 -> 0.34 T adds/s, fp64 0.043 -> 0.19.
        const int src = TB ? (l % 16) * 4 + l / 16 : l % (16 * V) / V * 4 + l / (16 * V) * V + l % V;
        bool own_col;
        const int col = col_at(l, own_col);
#pragma unroll
        for (int v = 0; v < VALS; ++v) {
            const int p = v0 + v;
            acc_t sum = 0;
#pragma unroll
            for (int s = 0; s < WK; ++s) sum += img[((s * NW + wg) * 4 + p % 4) * 256 + p / 4 * 64 + src];
            bool own_row;
            const int row = row_at(p, own_row);
            if (own_row && own_col) unsafeAtomicAdd(args.R + (int64_t)row * args.ldr + col, (T)sum);
        }
        return;
    }
#pragma unroll
    for (int v = 0; v < VALS; ++v) out[v] = 0;
#pragma unroll
    for (int s = 0; s < WK; ++s)
#pragma unroll
        for (int v = 0; v < VALS; ++v) out[v] += img[(((s * NW + wg) * 4 + (v0 + v) / 4) * 64 + l) * 4 + (v0 + v) % 4];
    typedef T uvec_raw __attribute__((ext_vector_type(U)));
    typedef uvec_raw uvec __attribute__((aligned(SZ)));
    bool own_r[VALS / U], own[VALS];
    T *dst[VALS];
    uvec old[VALS / U];
#pragma unroll
    for (int j = 0; j < VALS / U; ++j) {
        const int row = row_of(l, (v0 + j * U) / 4, own_r[j]);
        bool all = !TB && own_r[j];
#pragma unroll
        for (int e = 0; e < U; ++e) {
            bool oc;
            const int col = col_of(l, (v0 + j * U + e) % 4, oc);
            own[j * U + e] = own_r[j] && oc;
            all = all && oc;
            dst[j * U + e] = args.R + (int64_t)row * args.ldr + col;
        }
        own_r[j] = all;      // from here on: the U values go out as one access
        if (all) old[j] = *(const uvec *)dst[j * U];
    }
    // (edges after the whole pieces, so that only waves that have one wait between loads of one register)
#pragma unroll
    for (int j = 0; j < VALS / U; ++j)
#pragma unroll
        for (int e = 0; e < U; ++e)
            if (!own_r[j] && own[j * U + e]) old[j][e] = *dst[j * U + e];
#pragma unroll
    for (int j = 0; j < VALS / U; ++j) {
        if (own_r[j]) {
            uvec o = old[j];
#pragma unroll
            for (int e = 0; e < U; ++e) o[e] += (T)out[j * U + e];
            *(uvec *)dst[j * U] = o;
        } else {
#pragma unroll
            for (int e = 0; e < U; ++e) if (own[j * U + e]) *dst[j * U + e] = old[j][e] + (T)out[j * U + e];
        }
    }
}

template <typename T, int TASK, int TF, int TRANS, int WM, int WN, int WK, int NST, bool FAST>
static hipError_t launch_tile(int parts, const TileArgs<T> &args, hipStream_t s)
{
    constexpr int RING = tile_ring(WM, WN, WK, NST), SUMS = tile_sums(sizeof(T), WM, WN, WK);
    constexpr int LDS = RING > SUMS ? RING : SUMS;
    auto *const kernel = &mmlike_tile_kernel<T, TASK, TF, TRANS, WM, WN, WK, NST, FAST>;
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (granted != hipSuccess) return granted;
    const int64_t grid = xcd_grid((args.M + 16 * WM - 1) / (16 * WM), (args.N + 64 * WN - 1) / (64 * WN));
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    TileArgs<T> a = args;
    return launch_row_of_blocks(a, grid, 64 * WM * WN * WK, [&](unsigned n) {
        hipLaunchKernelGGL(kernel, dim3(n, (unsigned)parts), dim3(64 * WM * WN * WK), LDS, s, a);
    });
}

template <typename T, int TASK, int TF, int TRANS>
static hipError_t launch_tile_plan(const TilePlan &plan, const TileArgs<T> &a, hipStream_t s)
{
    constexpr bool FASTER = sizeof(T) == 4 && TASK == TASK_COUNT_GT && TF != THRES_ELEM;
    if constexpr (FASTER) {
        if (plan.us > COUNT_ROUNDING_TILE_US) {
            if (plan.wide) return launch_tile<T, TASK, TF, TRANS, 2, 1, 4, 3, true>(plan.parts, a, s);
            return launch_tile<T, TASK, TF, TRANS, 1, 1, 8, 2, true>(plan.parts, a, s);
        }
    }
    if (plan.wide) return launch_tile<T, TASK, TF, TRANS, 2, 1, 4, 3, false>(plan.parts, a, s);
    return launch_tile<T, TASK, TF, TRANS, 1, 1, 8, 2, false>(plan.parts, a, s);
}

template <typename T, int TASK, int TF>
static hipError_t launch_tile_layout(int trans, const TilePlan &plan, const TileArgs<T> &a, hipStream_t s)
{
    switch (trans) {
    case 0: return launch_tile_plan<T, TASK, TF, 0>(plan, a, s);
    case 1: return launch_tile_plan<T, TASK, TF, 1>(plan, a, s);
    case 2: return launch_tile_plan<T, TASK, TF, 2>(plan, a, s);
    default: return launch_tile_plan<T, TASK, TF, 3>(plan, a, s);
    }
}

template <typename T, int TASK>
hipError_t launch_mmlike_tile(int form, int trans, const TilePlan &plan, const TileArgs<T> &args, hipStream_t s)
{
    TileArgs<T> a = args;
    a.kpart = plan.kpart;
    a.kgroup = plan.kgroup;
    a.block_base = 0;
    switch (form) {
    case THRES_COL: return launch_tile_layout<T, TASK, THRES_COL>(trans, plan, a, s);
    case THRES_ROW: return launch_tile_layout<T, TASK, THRES_ROW>(trans, plan, a, s);
    case THRES_CONST: return launch_tile_layout<T, TASK, THRES_CONST>(trans, plan, a, s);
    default: return launch_tile_layout<T, TASK, THRES_ELEM>(trans, plan, a, s);
    }
}

}  // namespace amulet
#endif
