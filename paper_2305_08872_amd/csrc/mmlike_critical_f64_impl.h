// The predicate tasks in fp64 with fewer fp64 operations per product: DISCOUNT three instead of four and COUNT one and an fp32
// addition instead of two and two, by critical values; BOOST three instead of four, by a clamp.
//
// fl(a b) > th, th >= 0, is a >= c for b > 0 and a <= c for b < 0, with one critical value c per element of B and threshold
// that faces its column: rounding is monotonic.  (th < 0: fl(a b) > th unless fl(a (-b)) is more than the number below -th.)  c is
// found once per element as it is staged, for all rows of the tile, and then
//   t   = clamp((a - c') 2^300)        0 or 1, nothing between: c' is c or its neighbour, so that the difference is not 0
//   w   = base - t |cut|               the factor of a: b, or b (1 - dis)
//   acc = a w + acc
// with base = max(b, b (1 - dis)) and cut = b (1 - dis) - b: t is 1 where a product of a positive b is over its threshold, and where
// one of a negative b is not.  A product that is not over its threshold is added unrounded, one that is has its factor
// rounded instead of itself: no more error than rounding it.  That takes a cut that is exact, and so a 1 - dis of 0 or 1/2 to 1 (it would be off
// by half a last place of b, 1 / (1 - dis) times as much of the factor).  With others, masks: acc = a x + acc in the lanes where
// a > c' and acc = a y + acc in the others, x being b (1 - dis) for a positive b and y for a negative one; the other of them is
// b.  Three operations too, each term as exact, and as fast as the tile kernels' four (4096^3 7130 us by the clamp, 7690 by masks, tile
// kernels 7840).  A count has t = clamp(+-a 2^300 - |c'|), 1 over the threshold whatever
// b's sign, and adds t's high half as the fp32 number it also is, 15/8 or 0: fp32 additions issue from two waves at once, 32-bit ones
// of whole numbers do not (register-only, nominal clocks per 64 products: 7.2 so, 9.0 with v_add_u32 or any other).
// Thresholds of a count that face rows: the product of the transposed operands, transposed as it is added to R.
// BOOST's p + max(p - th, 0) is acc = a b' + acc and acc + clamp(a b' - th'), b' and th' being 2^-202 of b and th.
//
// A sum is added up in parts of a quarter of K, 64 k at most: an error as small as the tile kernels', whose waves share K
// (rms of 2^-53 of the terms' magnitudes, all of K in one sum / so / tile kernels: discount K = 8192 20.9 / 2.8 / 5.4, 256 3.8 / 1.1 / 1.1,
// boost 8192 1.6 / 0.20 / 0.46).  The sums' registers are those of operands read ahead: columns a k, rows a pair or two (all of
// them read as they are used: 2048^3 967 us).
//
// What bounds it: fp64 issue.  A register-only loop of the discount's three takes 12.8 clocks (at 2.4 GHz; the clock falls) per 64 products,
// of the four operations with their execution mask 18.8, of BOOST's three 14.0 (four: 18.2); the kernels 15.8, 14.8 and, for the count,
// 8.6, of which finding c is 1.1 (rows of a tile share it: 1.9 with 64 rows, 64 x 128 being the better tile for a K too short to hide a
// large one's ends) and barrier, loads and LDS the rest.
// us, tile kernels / here: discount 2048^3 1006 / 897, 4096^3 7800 / 7140, B transposed 7790 / 7250, 4096 x 2048 x 64 92 / 82;
// boost 2048^3 963 / 850, 4096^3 7610 / 6640, per row 7720 / 6420; count 2048^3 727 / 586, 4096^3 5640 / 3760, 4096 x 2048 x 64 65 / 50,
// per row 719 / 631, 5590 / 4070, 66 / 57.
// Values that none of these takes, in every tile, 4096^3 (tile kernels 7850, 7890, 5670): discount 8900, boost 8400 and count 5900 where the first stage
// has them, 10 700, 10 200 and 6900 at a quarter of K, and 16 300, 15 300 and 9800 where only the last half has: a tile is looked at after its
// first stage, after 8, and after twice as many each time, and what is refused at the end has run twice.
// A goes through LDS and is read back by broadcast: through the scalar cache, 8 bytes of 64 rows at a time, 4096^3 took
// 12 200 us.  256 columns in 256 registers per wave, two waves to a SIMD: 8530.  Stages of 8 k instead of 16: 7440 (128 rows).
// BOOST's plain sum on the fp64 matrix cores: they and the vector unit take turns (17.2 clocks, 8.1 + 9.2).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amulet_internal.h"

#ifndef AMULET_MMLIKE_CRITICAL_F64_IMPL_H
#define AMULET_MMLIKE_CRITICAL_F64_IMPL_H

namespace amulet {

typedef double cd2 __attribute__((ext_vector_type(2)));
typedef uint32_t cu2 __attribute__((ext_vector_type(2)));
typedef cd2 cd2_any __attribute__((aligned(8)));

constexpr int C64_COLS = 128, C64_TM = 8, C64_BP = C64_COLS + 2;
// pairs of columns of a lane: the count's sums are of 32 bits
constexpr int c64_pairs(int task) { return task == TASK_COUNT_GT ? 2 : 1; }
constexpr int c64_rows(int task, int waves) { return C64_TM * c64_pairs(task) * waves; }
constexpr double C64_SCALE = 0x1p300;
// (2^-202: p - th is then below 1 wherever BOOST takes the operands)
constexpr double C64_BOOST_SCALE = 0x1p-202, C64_LEAST_BOOST_TH = 0x1p-400;
constexpr double C64_LEAST_TH = 0x1p-100, C64_MOST_TH = 0x1p100;
// more than a product of a discount's operands: |a| below 2^900, |b| below 2^100
constexpr double C64_PRODUCTS = 0x1p1000;

// NW waves: 8 (stages of 8 k, two workgroups to a compute unit) or, for the discount, 16 (16 k, one)
template <int TASK, int NW>
struct Critical64Lds {
    static constexpr int BK = NW;
    // what an element of B comes to: the discount's base, c and cut (or x, c and y); c; or b
    static constexpr int KINDS = TASK == TASK_DISCOUNT ? 3 : 1, C = TASK == TASK_DISCOUNT ? 1 : 0, CUT = 2 % KINDS;
    double b[2][KINDS][BK][C64_BP];
    double a[2][BK][c64_rows(TASK, NW) + 2];
    double th[C64_COLS], half[C64_COLS], od[C64_COLS];
};

// How a tile's terms are formed; CRITICAL_DONE: they have been.
enum CriticalWay { CRITICAL_DONE, BY_CLAMP, BY_MASKS, BY_CLAMP_TO_LAST, BY_OWN_OPERATIONS };
// DISCOUNT's masks, and BOOST's clamp with a test for K's end at each k, for thresholds below 0 and a K that is not whole stages (4096^2 x
// 4093 6750 us, 6630 without the test, tile kernels 7600)
constexpr CriticalWay c64_second_way(int task) { return task == TASK_DISCOUNT ? BY_MASKS : task == TASK_BOOST ? BY_CLAMP_TO_LAST : BY_OWN_OPERATIONS; }

// The critical value of b for th, times what th and half, half the distance to the next double, come with: -2^300 (for thresholds
// below 0 2^300), or 1 (MASKS).  a b rounds to more than th from the middle th + half on, a tie if the next double is even.  n = (th + half) / b to within 2^-19 of its last place: rcp is good to 2^-24,
// one step to 2^-48, and the second step's remainder is exact but for its own rounding.  So the first a over the threshold is
// n or the next one away from 0, which its own product tells; b > 0, or ANY: the one below it is wanted.
template <bool ANY, bool MASKS>
__device__ __forceinline__ double critical_value_f64(double b, double th, double half)
{
    const double r = __builtin_amdgcn_rcp(b);
    const double q = th * r;
    double e = __builtin_fma(-q, b, th);
    double n = __builtin_fma(e, r, q);
    e = __builtin_fma(-n, b, th);
    e += half;
    n = __builtin_fma(e, r, n);
    const uint64_t nb = __builtin_bit_cast(uint64_t, n), bb = __builtin_bit_cast(uint64_t, b), tb = __builtin_bit_cast(uint64_t, th);
    const int away = __builtin_fabs(n * b) > __builtin_fabs(th) ? 1 : 0;
    if constexpr (ANY) return __builtin_bit_cast(double, ((nb - (uint64_t)away) & ~(1ull << 63)) | ((bb ^ tb) & (1ull << 63)));
    return __builtin_bit_cast(double, nb + (int64_t)((int)((uint32_t)((bb ^ (MASKS ? tb : ~tb)) >> 63)) - away));
}

// The next way for a tile that this one does not take, with R as it was.
template <int TASK, int TF, int TRANS, int NW, CriticalWay WAY, typename Args>
__device__ __forceinline__ CriticalWay critical_tile_f64(const Args &args, const unsigned tid, Critical64Lds<TASK, NW> &L)
{
    typedef Critical64Lds<TASK, NW> Lds;
    constexpr bool PLAIN = WAY == BY_OWN_OPERATIONS, MASKS = WAY == BY_MASKS, TO_LAST = PLAIN || WAY == BY_CLAMP_TO_LAST;
    constexpr bool transA = (TRANS & 1) != 0, transB = (TRANS & 2) != 0;
    constexpr int PAIRS = c64_pairs(TASK), ROWS = c64_rows(TASK, NW), BK = NW;
    constexpr bool ROW_SCALARS = TASK == TASK_BOOST && TF == THRES_ROW, SWAPPED = TASK == TASK_COUNT_GT && TF == THRES_ROW;
    constexpr int AE = PAIRS * BK / 8;  // values of A a thread stages (and two of B)
    const int M = args.M, N = args.N, K = args.K;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (M + ROWS - 1) / ROWS, tiles_n = (N + C64_COLS - 1) / C64_COLS;
    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, tiles_m, tiles_n, tm, tn)) return CRITICAL_DONE;
    const int row0 = tm * ROWS, col0 = tn * C64_COLS;
    const double *__restrict__ Ag = args.A;
    const double *__restrict__ Bg = args.B;
    // (N >= 2: a pair of columns that would end past N is the last two)
    auto col_at = [&](int p, bool &own) {
        const int u = col0 + (p & ~1);
        const int col = (u < N - 2 ? u : N - 2) + (p & 1);
        own = col >= u;
        return col;
    };
    // a lane's columns: 2 at, 2 at + 1 of the tile, at = lane, or lane mod 32 and 64 columns on; its rows: 8 of the wave's from first_row on
    const int at = lane % (64 / PAIRS), first_row = wave * (C64_TM * PAIRS) + lane / (64 / PAIRS) * C64_TM;
    auto own_col = [&](int c) { return at * 2 + (c & 1) + (c >> 1) * 64; };
    bool own;
    constexpr int NT = ROW_SCALARS ? C64_TM : 2 * PAIRS;
    double th[NT], od[2 * PAIRS];
    bool fit = true, first = true, zeros = false;     // (what all but the last way, or the first, take)
    auto fits = [&](double &t) {
        if constexpr (TASK == TASK_BOOST) {
            // (above +inf or no number, nothing: the clamp takes both, and all from 2^-400 up.  A k past the last one is nothing times nothing: over a
            // threshold below 0)
            first = first && !(t < 0.0 && K % BK != 0);
            const double m = __builtin_fabs(t);
            fit = fit && (t == 0.0 || (m >= C64_LEAST_BOOST_TH && t >= -C64_MOST_TH) || !(t < __builtin_inf()));
            t *= -C64_BOOST_SCALE;
        } else {
            // (no product is above +inf or above no number: no critical value, or, discounting, nothing taken off whatever it is.  A
            // discount's products are below 2^1000: none is over a threshold from there on, and all are over one from -2^1000 down,
            // whose critical value, infinite, masks take)
            const bool none = !(t < (TASK == TASK_DISCOUNT ? C64_PRODUCTS : __builtin_inf()));
            const bool always = TASK == TASK_DISCOUNT && t <= -C64_PRODUCTS;
            const double m = __builtin_fabs(t);
            zeros = zeros || t == 0.0;
            fit = fit && (none || always || t == 0.0 || (m >= C64_LEAST_TH && m <= C64_MOST_TH));
            if (none) t = TASK == TASK_DISCOUNT ? 1.0 : __builtin_nan("");
            // (a b > -m unless a -b > the number below m)
            if (t < 0.0) t = -__builtin_bit_cast(double, __builtin_bit_cast(uint64_t, m) - 1);
            if (always) t = -__builtin_inf();
            first = first && !always;
            t += 0.0;
            return none;
        }
        return false;
    };
    if constexpr (ROW_SCALARS) {
        // (the tile's 64 rows looked at by every wave, then its own)
        const int row = row0 + lane;
        double t = args.thres[row < M ? row : M - 1];
        if constexpr (!PLAIN) fits(t);
#pragma unroll
        for (int r = 0; r < C64_TM; ++r) {
            const int own_row = row0 + wave * C64_TM + r;
            th[r] = args.thres[own_row < M ? own_row : M - 1];
            const cu2 t = __builtin_bit_cast(cu2, PLAIN ? th[r] : th[r] * -C64_BOOST_SCALE);
            th[r] = __builtin_bit_cast(double, cu2{(uint32_t)__builtin_amdgcn_readfirstlane(t.x), (uint32_t)__builtin_amdgcn_readfirstlane(t.y)});
        }
    } else {
#pragma unroll
        for (int j = 0; j < 2 * PAIRS; ++j) {
            const int col = col_at(own_col(j), own);
            th[j] = args.thres[TF == THRES_CONST ? 0 : col];
            bool none = false;
            if constexpr (!PLAIN) none = fits(th[j]);
            if constexpr (TASK == TASK_DISCOUNT) {
                od[j] = 1.0 - args.dis[col];
                if (none) od[j] = 1.0;
                if constexpr (!PLAIN) fit = fit && __builtin_fabs(od[j]) <= C64_MOST_TH;
                first = first && (od[j] == 0.0 || (od[j] >= 0.5 && od[j] <= 1.0));
            }
        }
    }
    // (all waves face the same columns)
    if (!PLAIN && __builtin_amdgcn_ballot_w64(!fit) != 0) return BY_OWN_OPERATIONS;
    if (TASK != TASK_COUNT_GT && WAY == BY_CLAMP && __builtin_amdgcn_ballot_w64(!first) != 0) return c64_second_way(TASK);
    zeros = __builtin_amdgcn_ballot_w64(zeros) != 0;
    if constexpr (!PLAIN && TASK != TASK_BOOST) {
        if (wave == 0)
#pragma unroll
            for (int j = 0; j < 2 * PAIRS; ++j) {
                L.th[own_col(j)] = th[j] * (MASKS ? 1.0 : -C64_SCALE);
                L.half[own_col(j)] = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, th[j]) & 0xfff0000000000000ull) * (MASKS ? 0x1p-53 : -0x1p247);
                if constexpr (TASK == TASK_DISCOUNT) L.od[own_col(j)] = od[j];
            }
        __syncthreads();
    }
    // staging of B: one k of two neighbouring columns, or transposed one column's (and the 64th after it) by k
    auto place_b = [&](int x, int &k, int &c) { k = transB ? x % BK : wave; c = transB ? x / BK : (x & 63) * 2; };
    int bk, bc;
    place_b((int)tid, bk, bc);
    const int bcol = col_at(bc, own);
    const double *bsrc = transB ? Bg + (int64_t)bcol * args.ldb + bk : Bg + (int64_t)bk * args.ldb + bcol;
    const int bnext = transB ? (col_at(bc + 64, own) - bcol) * (int)args.ldb : 1;
    // and of A: AE neighbouring k of a row, or transposed AE k of a row, BK / AE apart
    auto place_a = [&](int x, int &k, int &row) { row = transA ? x % ROWS : x / (BK / AE); k = transA ? x / ROWS : x % (BK / AE) * AE; };
    int ak, arow;
    place_a((int)tid, ak, arow);
    const int arow_in = row0 + arow < M ? row0 + arow : M - 1;
    const double *asrc = transA ? Ag + (int64_t)ak * args.lda + arow_in : Ag + (int64_t)arow_in * args.lda + ak;
    constexpr int ASTEP = transA ? BK / AE : 1;
    // (the places computed again where they are used: held through the K loop they are registers too many)
    auto thread_again = [&] {
        int x = wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(x));
        return x;
    };
    uint64_t bad = 0;      // lanes that staged a value out of range
    float most = 0.0f;     // the largest high half of A's values
    constexpr float MOST_A = __builtin_bit_cast(float, (1023u + 900u) << 20);
    double sb[2], sa[AE];
    auto load = [&](int left) {      // `left` k of the range from this stage on
        if (left >= BK) {
            if constexpr (transB) {
                sb[0] = bsrc[0];
                sb[1] = bsrc[bnext];
            } else {
                const cd2 v = *(const cd2_any *)bsrc;
                sb[0] = v[0]; sb[1] = v[1];
            }
            if constexpr (AE == 2 && !transA) {
                const cd2 v = *(const cd2_any *)asrc;
                sa[0] = v[0]; sa[1] = v[1];
            } else {
#pragma unroll
                for (int i = 0; i < AE; ++i) sa[i] = asrc[(BK / AE) * i * args.lda];
            }
        } else {
            // a k past the last one: nothing times nothing (the plain way stops before it)
            int last = left - 1, ak, arow, bk, bc;
            asm volatile("" : "+s"(last));
            const int x = thread_again();
            place_a(x, ak, arow);
            place_b(x, bk, bc);
            auto at = [&](int k) { return k < last ? k : last; };
            const double *from = bsrc + (int64_t)(at(bk) - bk) * (transB ? 1 : args.ldb);
            const double b0 = from[0], b1 = from[bnext];
            sb[0] = bk <= last ? b0 : 0.0;
            sb[1] = bk <= last ? b1 : 0.0;
#pragma unroll
            for (int i = 0; i < AE; ++i) {
                const int k = ak + ASTEP * i;
                const double v = asrc[(int64_t)(at(k) - ak) * (transA ? args.lda : 1)];
                sa[i] = k <= last ? v : 0.0;
            }
        }
        bsrc += transB ? (int64_t)BK : (int64_t)BK * args.ldb;
        asrc += transA ? (int64_t)BK * args.lda : (int64_t)BK;
    };
    auto store = [&](int buf) {
        int ak, arow, bk, bc;
        const int x = thread_again();
        place_a(x, ak, arow);
        place_b(x, bk, bc);
#pragma unroll
        for (int i = 0; i < AE; ++i) L.a[buf][ak + ASTEP * i][arow] = !PLAIN && TASK == TASK_COUNT_GT ? sa[i] * (C64_SCALE / 2) : sa[i];
        double c[2], base[2], cut[2];
        bool in = true;
        // |a| and |b| from 2^-400 to below 2^100, or 0
        auto boost_takes = [](double v) {
            const uint32_t top = (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32) & 0x7fffffffu;
            constexpr uint32_t LEAST = (1023u - 400u) << 20, MOST = (1023u + 100u) << 20;
            return top - LEAST < MOST - LEAST || v == 0.0;
        };
        if constexpr (!PLAIN && TASK == TASK_BOOST) {
#pragma unroll
            for (int i = 0; i < AE; ++i) in = in && boost_takes(sa[i]);
        } else if constexpr (!PLAIN && TASK == TASK_DISCOUNT) {
            // (|a| below 2^900: with |b| below 2^100 no product is past the largest double, which would be infinite before the discount
            // is taken off.  High halves as fp32 numbers come in the same order, and then no numbers, which a maximum keeps)
            auto high = [](double v) { return __builtin_bit_cast(float, (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32)); };
            // (B transposed, there is no register for the largest: looked at each time)
            if constexpr (transB) most = 0.0f;
            asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(high(sa[0])), "v"(high(sa[AE - 1])));
            if constexpr (transB) in = in && most < MOST_A;
        }
        if (!PLAIN && TASK != TASK_BOOST && zeros) {
            // (a threshold of 0 has 0 for its critical value, as no product is rounded to 0: |a| of 2^-299 or more, or 0)
#pragma unroll
            for (int i = 0; i < AE; ++i) in = in && (__builtin_fabs(sa[i]) >= 0x1p-299 || sa[i] == 0.0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int col = bc + (transB ? 64 * i : i);
            const double b = sb[i];
            base[i] = b;
            if constexpr (!PLAIN && TASK == TASK_BOOST) {
                base[i] = b * C64_BOOST_SCALE;
                in = in && boost_takes(b);
            } else if constexpr (!PLAIN) {
                // |b| from 2^-600 to below 2^100, or 0 (whose base and cut are 0 whatever its c, which is not a number): with th of
                // 2^-100 to 2^100 c is 2^-200 to 2^700, and a distance of one last place of it times 2^300 more than 1
                const uint32_t top = (uint32_t)(__builtin_bit_cast(uint64_t, b) >> 32) & 0x7fffffffu;
                constexpr uint32_t LEAST = (1023u - 600u) << 20, MOST = (1023u + 100u) << 20;
                in = in && (top - LEAST < MOST - LEAST || b == 0.0);
                c[i] = critical_value_f64<TASK == TASK_COUNT_GT, MASKS>(b, L.th[col], L.half[col]);
                if constexpr (MASKS) c[i] = L.th[col] < -C64_PRODUCTS ? __builtin_copysign(__builtin_inf(), -b) : c[i];
                if constexpr (TASK == TASK_DISCOUNT) {
                    const double m = b * L.od[col];
                    if constexpr (MASKS) {
                        base[i] = b > 0.0 ? m : b;
                        cut[i] = b > 0.0 ? b : m;
                    } else {
                        asm("v_max_f64 %0, %1, %2" : "=v"(base[i]) : "v"(b), "v"(m));
                        cut[i] = m - b;
                    }
                }
            }
        }
        if constexpr (!PLAIN) bad |= __builtin_amdgcn_ballot_w64(!in);
        auto put = [&](double (&to)[BK][C64_BP], const double (&v)[2]) {
            if constexpr (transB) { to[bk][bc] = v[0]; to[bk][bc + 64] = v[1]; }
            else *(cd2 *)&to[bk][bc] = cd2{v[0], v[1]};
        };
        if constexpr (PLAIN || TASK != TASK_COUNT_GT) put(L.b[buf][0], base);
        if constexpr (!PLAIN && TASK != TASK_BOOST) put(L.b[buf][Lds::C], c);
        if constexpr (!PLAIN && TASK == TASK_DISCOUNT) put(L.b[buf][Lds::CUT], cut);
    };
    auto refused = [&] { return __syncthreads_or(bad != 0 || (!transB && !(most < MOST_A))) != 0; };

    typedef typename std::conditional<TASK == TASK_COUNT_GT, uint32_t, double>::type sum_t;
    sum_t acc[C64_TM][2 * PAIRS];
#pragma unroll
    for (int r = 0; r < C64_TM; ++r)
#pragma unroll
        for (int c = 0; c < 2 * PAIRS; ++c) acc[r][c] = 0;
    double big = C64_SCALE;
    asm volatile("" : "+s"(big));
    const uint64_t active = __builtin_amdgcn_read_exec();
    struct Columns { cd2 b[PAIRS], c, cut; };
    auto columns_of = [&](int buf, int k) {
        Columns o;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) o.b[p] = *(const cd2 *)&L.b[buf][0][k][at * 2 + 64 * p];
        if constexpr (!PLAIN && TASK == TASK_DISCOUNT) { o.c = *(const cd2 *)&L.b[buf][Lds::C][k][at * 2]; o.cut = *(const cd2 *)&L.b[buf][Lds::CUT][k][at * 2]; }
        return o;
    };
    auto rows_of = [&](int buf, int k, int pair) { return *(const cd2 *)&L.a[buf][k][first_row + 2 * pair]; };
    auto th_of = [&](int r, int c) { return th[ROW_SCALARS ? r : c]; };
    // 2 with the sign of the critical value of a column (A has the rest of 2^300): an operand that an instruction can hold
    cu2 sgn[2 * PAIRS];
#pragma unroll
    for (int c = 0; c < 2 * PAIRS; ++c) sgn[c] = cu2{0, 0};
    uint32_t sign = 0x80000000u;
    asm volatile("" : "+s"(sign));
    // a column's products with a pair of rows
    auto fold = [&](const Columns &o, const cd2 &rows, int r) {
        if constexpr (TASK == TASK_COUNT_GT && !PLAIN)
            if (r == 0)
#pragma unroll
                for (int c = 0; c < 2 * PAIRS; ++c)
                    sgn[c].y = ((uint32_t)(__builtin_bit_cast(uint64_t, (double)o.b[c / 2][c & 1]) >> 32) & sign) | 0x40000000u;
        {
            const double a = rows[0], e = rows[1];
            double t[4];
            if constexpr (TASK == TASK_DISCOUNT && PLAIN) {
                // (four comparisons first: each followed by its own masked product, as in mmlike_valu_f64.hip, 4096^3 9220 us, so 8865)
                uint64_t over[4];
                asm volatile("v_mul_f64 %0, %[a], %[b0]\n\tv_mul_f64 %1, %[a], %[b1]\n\tv_mul_f64 %2, %[e], %[b0]\n\tv_mul_f64 %3, %[e], %[b1]\n\t"
                             "v_cmp_gt_f64_e64 %8, %0, %[th0]\n\tv_cmp_gt_f64_e64 %9, %1, %[th1]\n\tv_cmp_gt_f64_e64 %10, %2, %[th0]\n\tv_cmp_gt_f64_e64 %11, %3, %[th1]\n\t"
                             "s_mov_b64 exec, %8\n\tv_mul_f64 %0, %0, %[od0]\n\ts_mov_b64 exec, %9\n\tv_mul_f64 %1, %1, %[od1]\n\t"
                             "s_mov_b64 exec, %10\n\tv_mul_f64 %2, %2, %[od0]\n\ts_mov_b64 exec, %11\n\tv_mul_f64 %3, %3, %[od1]\n\ts_mov_b64 exec, %[active]\n\t"
                             "v_add_f64 %4, %4, %0\n\tv_add_f64 %5, %5, %1\n\tv_add_f64 %6, %6, %2\n\tv_add_f64 %7, %7, %3"
                             : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1]),
                               "=&s"(over[0]), "=&s"(over[1]), "=&s"(over[2]), "=&s"(over[3])
                             : [a] "v"(a), [e] "v"(e), [b0] "v"(o.b[0][0]), [b1] "v"(o.b[0][1]), [th0] "v"(th[0]), [th1] "v"(th[1]), [od0] "v"(od[0]), [od1] "v"(od[1]), [active] "s"(active));
            } else if constexpr (TASK == TASK_DISCOUNT && MASKS) {
#define AMULET_EITHER(SUM, MASK, A, X, Y) "s_mov_b64 exec, " MASK "\n\tv_fma_f64 " SUM ", " A ", " X ", " SUM "\n\ts_xor_b64 exec, exec, %[active]\n\tv_fma_f64 " SUM ", " A ", " Y ", " SUM "\n\t"
                uint64_t over[4];
                asm volatile("v_cmp_gt_f64_e64 %4, %[a], %[c0]\n\tv_cmp_gt_f64_e64 %5, %[a], %[c1]\n\tv_cmp_gt_f64_e64 %6, %[e], %[c0]\n\tv_cmp_gt_f64_e64 %7, %[e], %[c1]\n\t"
                             AMULET_EITHER("%0", "%4", "%[a]", "%[x0]", "%[y0]") AMULET_EITHER("%1", "%5", "%[a]", "%[x1]", "%[y1]")
                             AMULET_EITHER("%2", "%6", "%[e]", "%[x0]", "%[y0]") AMULET_EITHER("%3", "%7", "%[e]", "%[x1]", "%[y1]") "s_mov_b64 exec, %[active]"
                             : "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1]), "=&s"(over[0]), "=&s"(over[1]), "=&s"(over[2]), "=&s"(over[3])
                             : [a] "v"(a), [e] "v"(e), [c0] "v"(o.c[0]), [c1] "v"(o.c[1]), [x0] "v"(o.b[0][0]), [x1] "v"(o.b[0][1]), [y0] "v"(o.cut[0]), [y1] "v"(o.cut[1]), [active] "s"(active)
                             : "scc");
#undef AMULET_EITHER
            } else if constexpr (TASK == TASK_DISCOUNT) {
                asm volatile("v_fma_f64 %0, %8, %10, %11 clamp\n\tv_fma_f64 %1, %8, %10, %12 clamp\n\tv_fma_f64 %2, %9, %10, %11 clamp\n\tv_fma_f64 %3, %9, %10, %12 clamp\n\t"
                             "v_fma_f64 %0, %0, -|%13|, %15\n\tv_fma_f64 %1, %1, -|%14|, %16\n\tv_fma_f64 %2, %2, -|%13|, %15\n\tv_fma_f64 %3, %3, -|%14|, %16\n\t"
                             "v_fma_f64 %4, %8, %0, %4\n\tv_fma_f64 %5, %8, %1, %5\n\tv_fma_f64 %6, %9, %2, %6\n\tv_fma_f64 %7, %9, %3, %7"
                             : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1])
                             : "v"(a), "v"(e), "s"(big), "v"(o.c[0]), "v"(o.c[1]), "v"(o.cut[0]), "v"(o.cut[1]), "v"(o.b[0][0]), "v"(o.b[0][1]));
            } else if constexpr (TASK == TASK_BOOST) {
#define AMULET_BOOST_F64(TH, TAKE, TOP) \
                asm volatile("v_fma_f64 %0, %8, %10, " TH "%12" TAKE "v_fma_f64 %1, %8, %11, " TH "%13" TAKE "v_fma_f64 %2, %9, %10, " TH "%14" TAKE "v_fma_f64 %3, %9, %11, " TH "%15" TAKE \
                             "v_fma_f64 %4, %8, %10, %4\n\tv_fma_f64 %5, %8, %11, %5\n\tv_fma_f64 %6, %9, %10, %6\n\tv_fma_f64 %7, %9, %11, %7\n\t" TOP \
                             "v_add_f64 %4, %4, %0\n\tv_add_f64 %5, %5, %1\n\tv_add_f64 %6, %6, %2\n\tv_add_f64 %7, %7, %3" \
                             : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1]) \
                             : "v"(a), "v"(e), "v"(o.b[0][0]), "v"(o.b[0][1]), AMULET_TH(th_of(r, 0)), AMULET_TH(th_of(r, 1)), AMULET_TH(th_of(r + 1, 0)), AMULET_TH(th_of(r + 1, 1)))
#define AMULET_BOOST_F64_WAYS \
                if constexpr (PLAIN) AMULET_BOOST_F64("-", "\n\t", "v_max_f64 %0, %0, 0\n\tv_max_f64 %1, %1, 0\n\tv_max_f64 %2, %2, 0\n\tv_max_f64 %3, %3, 0\n\t"); \
                else AMULET_BOOST_F64("", " clamp\n\t", "")
                // (thresholds that face rows are the same for the wave: scalar registers)
                if constexpr (TF == THRES_ROW) {
#define AMULET_TH "s"
                    AMULET_BOOST_F64_WAYS;
#undef AMULET_TH
                } else {
#define AMULET_TH "v"
                    AMULET_BOOST_F64_WAYS;
#undef AMULET_TH
                }
#undef AMULET_BOOST_F64_WAYS
#undef AMULET_BOOST_F64
            } else if constexpr (PLAIN) {
#pragma unroll
                for (int p = 0; p < PAIRS; ++p)
                    asm volatile("v_mul_f64 v[124:125], %4, %6\n\tv_mul_f64 v[126:127], %4, %7\n\t"
                                 "v_cmp_gt_f64_e32 vcc, v[124:125], %8\n\tv_addc_co_u32_e32 %0, vcc, 0, %0, vcc\n\tv_mul_f64 v[124:125], %5, %6\n\t"
                                 "v_cmp_gt_f64_e32 vcc, v[126:127], %9\n\tv_addc_co_u32_e32 %1, vcc, 0, %1, vcc\n\tv_mul_f64 v[126:127], %5, %7\n\t"
                                 "v_cmp_gt_f64_e32 vcc, v[124:125], %8\n\tv_addc_co_u32_e32 %2, vcc, 0, %2, vcc\n\tv_cmp_gt_f64_e32 vcc, v[126:127], %9\n\tv_addc_co_u32_e32 %3, vcc, 0, %3, vcc"
                                 : "+v"(acc[r][2 * p]), "+v"(acc[r][2 * p + 1]), "+v"(acc[r + 1][2 * p]), "+v"(acc[r + 1][2 * p + 1])
                                 : "v"(a), "v"(e), "v"(o.b[p][0]), "v"(o.b[p][1]), "v"(th[2 * p]), "v"(th[2 * p + 1])
                                 : "vcc", "v124", "v125", "v126", "v127");
            } else {
#pragma unroll
                for (int p = 0; p < PAIRS; ++p)
                    asm volatile("v_fma_f64 v[120:121], %4, -%6, -|%8| clamp\n\tv_fma_f64 v[122:123], %4, -%7, -|%9| clamp\n\t"
                                 "v_fma_f64 v[124:125], %5, -%6, -|%8| clamp\n\tv_fma_f64 v[126:127], %5, -%7, -|%9| clamp\n\t"
                                 "v_add_f32 %0, %0, v121\n\tv_add_f32 %1, %1, v123\n\tv_add_f32 %2, %2, v125\n\tv_add_f32 %3, %3, v127"
                                 : "+v"(acc[r][2 * p]), "+v"(acc[r][2 * p + 1]), "+v"(acc[r + 1][2 * p]), "+v"(acc[r + 1][2 * p + 1])
                                 : "v"(a), "v"(e), "v"(sgn[2 * p]), "v"(sgn[2 * p + 1]), "v"(o.b[p][0]), "v"(o.b[p][1])
                                 : "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127");
            }
        }
    };
    // Sums of a quarter of K, 64 k at most, are added up on their own: the rounding of one running sum grows with its length.
    double all[C64_TM][2];
    const int every = K / 4 <= BK ? 1 : K / 4 < 64 ? K / 4 / BK : 64 / BK;
    int until = every;
    auto gather = [&] {
        until = every;
#pragma unroll
        for (int r = 0; r < C64_TM; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) { all[r][c] += acc[r][c]; acc[r][c] = 0; }
    };
    if constexpr (TASK != TASK_COUNT_GT)
#pragma unroll
        for (int r = 0; r < C64_TM; ++r) all[r][0] = all[r][1] = 0.0;
    // (operands ahead: those of the next k's columns, and of AHEAD pairs of rows)
    constexpr int HALF = C64_TM / 2, AHEAD = TASK == TASK_COUNT_GT ? HALF : TASK == TASK_BOOST ? 2 : 1, RING = 2 * AHEAD;
    Columns o[2];
    cd2 rows[RING];
    const int stages = (K + BK - 1) / BK;
    load(K);
    store(0);
    if (PLAIN) __syncthreads();
    else if (refused()) return BY_OWN_OPERATIONS;
    for (int t = 0; t < stages; ++t) {
        const int buf = t & 1, k0 = t * BK;
        if (t + 1 < stages) load(K - (t + 1) * BK);
        // (the plain way in eights, so that its loop is unrolled, and to the last k)
#pragma unroll
        for (int h = 0; h < BK; h += 8) {
            if (TO_LAST && k0 + h >= K) break;
            if (PLAIN || h == 0) {
                o[0] = columns_of(buf, h);
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) rows[i] = rows_of(buf, h, i);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (TO_LAST && k0 + h + k >= K) break;
                const bool more = k < 7 || (!PLAIN && h + 8 < BK);
#pragma unroll
                for (int i = 0; i < HALF; ++i) {
                    const int at_row = k * HALF + i, next = at_row + AHEAD;
                    if (i == 0 && more) o[(k + 1) & 1] = columns_of(buf, h + k + 1);
                    if (next < (k + 1) * HALF || more) rows[next % RING] = rows_of(buf, h + next / HALF, next % HALF);
                    __builtin_amdgcn_sched_barrier(0);
                    fold(o[k & 1], rows[at_row % RING], 2 * i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (TASK != TASK_COUNT_GT)
            if (--until == 0) gather();
        if (t + 1 < stages) store(buf ^ 1);
        // (looked at after the first stage, some 64 or 128 k, and twice as many each time, and at the end)
        if (!PLAIN && (t & (t + 1)) == 0 && t >= 7) {
            if (refused()) return BY_OWN_OPERATIONS;
        } else __syncthreads();
    }
    if (!PLAIN && refused()) return BY_OWN_OPERATIONS;
    if constexpr (TASK != TASK_COUNT_GT) gather();

    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    const int wrow = row0 + wave * (C64_TM * PAIRS) + l / (64 / PAIRS) * C64_TM;
    bool below[2] = {false, false};     // (a negative threshold: what was counted are the others)
    auto sum = [&](int r, int c) {
        if constexpr (TASK == TASK_COUNT_GT && PLAIN) return (double)acc[r][c];
        else if constexpr (TASK == TASK_COUNT_GT) {
            const int n = (int)((uint32_t)(__builtin_bit_cast(float, acc[r][c]) * 8.0f) / 15u);
            return (double)(below[c & 1] ? K - n : n);
        }
        else return TASK == TASK_BOOST && !PLAIN ? all[r][c] / C64_BOOST_SCALE : all[r][c];
    };
    if constexpr (SWAPPED) {
        // (a lane's eight rows lie next to each other in R)
#pragma unroll
        for (int j = 0; j < 2 * PAIRS; ++j) {
            const int col = col_at(l % (64 / PAIRS) * 2 + (j & 1) + 64 * (j >> 1), own);
            below[j & 1] = !PLAIN && args.thres[col] < 0.0;
            double *const dst = args.R + (int64_t)col * args.ldr + wrow;
            if (!own) continue;
            if (wrow + C64_TM <= M) {
                cd2 old[C64_TM / 2];
#pragma unroll
                for (int r = 0; r < C64_TM / 2; ++r) old[r] = *(const cd2_any *)(dst + 2 * r);
#pragma unroll
                for (int r = 0; r < C64_TM / 2; ++r) *(cd2_any *)(dst + 2 * r) = old[r] + cd2{sum(2 * r, j), sum(2 * r + 1, j)};
            } else {
#pragma unroll
                for (int r = 0; r < C64_TM; ++r)
                    if (wrow + r < M) dst[r] += sum(r, j);
            }
        }
        return CRITICAL_DONE;
    }
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        cd2 old[C64_TM];
        bool last, whole;
        const int tcol = l % (64 / PAIRS) * 2 + 64 * p, col = col_at(tcol, whole);
        (void)col_at(tcol + 1, last);
        whole = whole && last;
        if constexpr (TASK == TASK_COUNT_GT && !PLAIN)
            for (int c = 0; c < 2; ++c) below[c] = args.thres[TF == THRES_CONST ? 0 : col_at(tcol + c, own)] < 0.0;
#pragma unroll
        for (int r = 0; r < C64_TM; ++r) {
            old[r] = cd2{0, 0};
            if (whole && wrow + r < M) old[r] = *(const cd2_any *)(args.R + (int64_t)(wrow + r) * args.ldr + col);
        }
#pragma unroll
        for (int r = 0; r < C64_TM; ++r) {
            if (wrow + r >= M) break;
            double *const dst_row = args.R + (int64_t)(wrow + r) * args.ldr;
            if (whole) *(cd2_any *)(dst_row + col) = old[r] + cd2{sum(r, 2 * p), sum(r, 2 * p + 1)};
            else
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int to = col_at(tcol + c, own);
                    if (own) dst_row[to] += sum(r, 2 * p + c);
                }
        }
    }
    return CRITICAL_DONE;
}

// A tile by critical values, or, if it holds what they do not take, by the task's own operations.
template <int TASK, int TF, int TRANS, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
mmlike_critical_f64_kernel(const MmlikeArgsF64 args)
{
    extern __shared__ __attribute__((aligned(16))) char critical64_smem[];
    Critical64Lds<TASK, NW> &L = *(Critical64Lds<TASK, NW> *)critical64_smem;
    const unsigned wave = own_wave();
    const CriticalWay way = critical_tile_f64<TASK, TF, TRANS, NW, BY_CLAMP>(args, threadIdx.x, L);
    if (way == CRITICAL_DONE) return;
    unsigned tid;
    if constexpr (TASK != TASK_COUNT_GT)
        if (way != BY_OWN_OPERATIONS) {
            const auto &again = opaque_args<MmlikeArgsF64>(wave, tid);
            if (critical_tile_f64<TASK, TF, TRANS, NW, c64_second_way(TASK)>(again, tid, L) == CRITICAL_DONE) return;
        }
    const auto &again = opaque_args<MmlikeArgsF64>(wave, tid);
    critical_tile_f64<TASK, TF, TRANS, NW, BY_OWN_OPERATIONS>(again, tid, L);
}

template <int TASK, int TF, int TRANS, int NW>
static hipError_t launch_critical_f64(const MmlikeArgsF64 &args, hipStream_t s)
{
    constexpr int ROWS = c64_rows(TASK, NW), LDS_BYTES = (int)sizeof(Critical64Lds<TASK, NW>);
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&mmlike_critical_f64_kernel<TASK, TF, TRANS, NW>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (granted != hipSuccess) return granted;
    MmlikeArgsF64 b = args;
    const int64_t blocks = xcd_grid(((int64_t)b.M + ROWS - 1) / ROWS, ((int64_t)b.N + C64_COLS - 1) / C64_COLS);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    return launch_row_of_blocks(b, blocks, 64 * NW, [&](unsigned n) {
        hipLaunchKernelGGL((mmlike_critical_f64_kernel<TASK, TF, TRANS, NW>), dim3(n), dim3(64 * NW), LDS_BYTES, s, b);
    });
}

template <int TASK, int TF, int NW>
static hipError_t launch_critical_f64(const MmlikeArgsF64 &a, hipStream_t s)
{
    switch ((a.transA ? 1 : 0) | (a.transB ? 2 : 0)) {
    case 0: return launch_critical_f64<TASK, TF, 0, NW>(a, s);
    case 1: return launch_critical_f64<TASK, TF, 1, NW>(a, s);
    case 2: return launch_critical_f64<TASK, TF, 2, NW>(a, s);
    default: return launch_critical_f64<TASK, TF, 3, NW>(a, s);
    }
}

template <int TASK, int TF>
hipError_t launch_mmlike_critical_f64(const MmlikeArgsF64 &a, int rows, hipStream_t s)
{
    if constexpr (TASK == TASK_DISCOUNT)
        if (rows == 128) return launch_critical_f64<TASK, TF, 16>(a, s);
    return launch_critical_f64<TASK, TF, 8>(a, s);
}

}  // namespace amulet
#endif
