// DISCOUNT in fp64 by critical values: three fp64 operations per product instead of four.
//
// fl(a b) > th, th > 0, is a >= c for b > 0 and a <= c for b < 0, with one critical value c per element of B and threshold
// that faces its column: rounding is monotonic.  c is found once per element as it is staged, for all rows of the tile, and then
//   t   = clamp((a - c') 2^300)        0 or 1, nothing between: c' is c or its neighbour, so that the difference is not 0
//   w   = base - t |cut|               the factor of a: b, or b (1 - dis)
//   acc = a w + acc
// with base = max(b, b (1 - dis)) and cut = b (1 - dis) - b: t is 1 where a product of a positive b is over its threshold, and where
// one of a negative b is not.  A product that is not over its threshold is added unrounded, one that is has its factor
// rounded instead of itself: no more error than rounding it.
//
// What bounds it: fp64 issue.  A register-only loop of the three takes 12.8 clocks (at 2.4 GHz) per 64 products, of the four operations with
// their execution mask 18.8; this kernel 15.2 at 2048^3 and 4096^3, of which finding c is 1.1 (rows of a tile share it: 1.9 with 64
// rows, 64 x 128 being the better tile for a K too short to hide a large one's ends) and barrier, loads and LDS the rest; at 2.25 GHz.
// us, tile kernels / here: 2048^3 1012 / 887, 4096^3 7810 / 6930, A transposed 7930 / 7030, B transposed 7790 / 7120,
// 2496 x 896 x 6601 1865 / 1640, 1142 x 5056 x 64 69 / 57.
// A goes through LDS and is read back by broadcast: through the scalar cache, 8 bytes of 64 rows at a time, 4096^3 took
// 12 200 us.  256 columns in 256 registers per wave, two waves to a SIMD: 8530.  Stages of 8 k instead of 16: 7440 (128 rows).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amulet_internal.h"

#ifndef AMULET_MMLIKE_CRITICAL_F64_IMPL_H
#define AMULET_MMLIKE_CRITICAL_F64_IMPL_H

namespace amulet {

typedef double cd2 __attribute__((ext_vector_type(2)));
typedef cd2 cd2_any __attribute__((aligned(8)));

constexpr int C64_COLS = 128, C64_TM = 8, C64_BP = C64_COLS + 2;
constexpr double C64_SCALE = 0x1p300;
constexpr double C64_LEAST_TH = 0x1p-100, C64_MOST_TH = 0x1p100;

// NW waves: 8 (64 rows, stages of 8 k, two workgroups to a compute unit) or 16 (128 rows, 16 k, one)
template <int NW>
struct Critical64Lds {
    static constexpr int BK = NW;
    double c[2][BK][C64_BP];
    double base[2][BK][C64_BP];
    double cut[2][BK][C64_BP];
    double a[2][BK][C64_TM * NW + 2];
    double th[C64_COLS], half[C64_COLS], od[C64_COLS];
};

// The critical value of b for th, times -2^300, as th and half, half the distance to the next double, come.  a b rounds to more than
// th from the middle th + half on, a tie if the next double is even.  n = (th + half) / b to within 2^-19 of its last place: rcp is good to 2^-24,
// one step to 2^-48, and the second step's remainder is exact but for its own rounding.  So the first a over the threshold is
// n or the next one away from 0, which its own product tells; b > 0: the one below it is wanted.
__device__ __forceinline__ double critical_value_f64(double b, double th, double half)
{
    const double r = __builtin_amdgcn_rcp(b);
    const double q = th * r;
    double e = __builtin_fma(-q, b, th);
    double n = __builtin_fma(e, r, q);
    e = __builtin_fma(-n, b, th);
    e += half;
    n = __builtin_fma(e, r, n);
    const double p = n * b;
    const uint64_t bits = __builtin_bit_cast(uint64_t, n);
    const int step = (int)((uint32_t)(__builtin_bit_cast(uint64_t, b) >> 63)) - (p < th ? 1 : 0);
    return __builtin_bit_cast(double, bits + (int64_t)step);
}

// PLAIN: the task's own four operations, for a tile that the first way gives back (false) with R as it was.
template <int TF, int TRANS, int NW, bool PLAIN, typename Args>
__device__ __forceinline__ bool critical_tile_f64(const Args &args, const unsigned tid, Critical64Lds<NW> &L)
{
    constexpr bool transA = (TRANS & 1) != 0, transB = (TRANS & 2) != 0;
    constexpr int ROWS = C64_TM * NW, BK = NW;
    constexpr int AE = BK / 8;          // values of A a thread stages (and two of B)
    const int M = args.M, N = args.N, K = args.K;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (M + ROWS - 1) / ROWS, tiles_n = (N + C64_COLS - 1) / C64_COLS;
    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, tiles_m, tiles_n, tm, tn)) return true;
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
    // a lane's columns: 2 lane, 2 lane + 1 of the tile
    bool own;
    double th[2], od[2];
    bool fit = true;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int col = col_at(lane * 2 + j, own);
        th[j] = args.thres[TF == THRES_CONST ? 0 : col];
        od[j] = 1.0 - args.dis[col];
        if constexpr (!PLAIN) {
            // (no product is above +inf or above no number: nothing is taken off, whatever the critical value)
            if (!(th[j] < __builtin_inf())) { th[j] = 1.0; od[j] = 1.0; }
            fit = fit && th[j] >= C64_LEAST_TH && th[j] <= C64_MOST_TH && od[j] >= 0.0 && od[j] <= 1.0;
        }
    }
    if (!PLAIN && __builtin_amdgcn_ballot_w64(!fit) != 0) return false;     // (all waves face the same columns)
    if constexpr (!PLAIN) {
        if (wave == 0)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                L.th[lane * 2 + j] = th[j] * -C64_SCALE;
                L.half[lane * 2 + j] = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, th[j]) & 0x7ff0000000000000ull) * -0x1p247;
                L.od[lane * 2 + j] = od[j];
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
    // and of A: AE neighbouring k of a row, or transposed one k (and the 8th after it) of a row
    auto place_a = [&](int x, int &k, int &row) { row = transA ? x % ROWS : x >> 3; k = transA ? x / ROWS : (x & 7) * AE; };
    int ak, arow;
    place_a((int)tid, ak, arow);
    const int arow_in = row0 + arow < M ? row0 + arow : M - 1;
    const double *asrc = transA ? Ag + (int64_t)ak * args.lda + arow_in : Ag + (int64_t)arow_in * args.lda + ak;
    constexpr int ASTEP = transA ? 8 : 1;
    uint64_t bad = 0;      // lanes that staged a value of B out of range
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
                for (int i = 0; i < AE; ++i) sa[i] = asrc[8 * i * args.lda];
            }
        } else {
            // a k past the last one: nothing times nothing (the plain way stops before it)
            int last = left - 1;
            asm volatile("" : "+s"(last));
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
        // (the places in LDS computed again: held through the K loop they are registers too many)
        int x = wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), ak, arow, bk, bc;
        asm volatile("" : "+v"(x));
        place_a(x, ak, arow);
        place_b(x, bk, bc);
#pragma unroll
        for (int i = 0; i < AE; ++i) L.a[buf][ak + ASTEP * i][arow] = sa[i];
        double c[2], base[2], cut[2];
        bool in = true;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int col = bc + (transB ? 64 * i : i);
            const double b = sb[i];
            base[i] = b;
            if constexpr (!PLAIN) {
                // |b| of 2^-600 to 2^101, or 0 (whose base and cut are 0 whatever its c, which is not a number): with th of
                // 2^-100 to 2^100 c is 2^-201 to 2^700, and a distance of one last place of it times 2^300 more than 1
                const uint32_t top = (uint32_t)(__builtin_bit_cast(uint64_t, b) >> 32) & 0x7fffffffu;
                constexpr uint32_t LEAST = (1023u - 600u) << 20, MOST = (1023u + 100u) << 20;
                in = in && (top - LEAST <= MOST - LEAST || b == 0.0);
                c[i] = critical_value_f64(b, L.th[col], L.half[col]);
                const double m = b * L.od[col];
                asm("v_max_f64 %0, %1, %2" : "=v"(base[i]) : "v"(b), "v"(m));
                cut[i] = m - b;
            }
        }
        if constexpr (!PLAIN) bad |= __builtin_amdgcn_ballot_w64(!in);
        auto put = [&](double (&to)[BK][C64_BP], const double (&v)[2]) {
            if constexpr (transB) { to[bk][bc] = v[0]; to[bk][bc + 64] = v[1]; }
            else *(cd2 *)&to[bk][bc] = cd2{v[0], v[1]};
        };
        put(L.base[buf], base);
        if constexpr (!PLAIN) { put(L.c[buf], c); put(L.cut[buf], cut); }
    };
    auto refused = [&] { return __syncthreads_or(bad != 0) != 0; };

    double acc[C64_TM][2];
#pragma unroll
    for (int r = 0; r < C64_TM; ++r) acc[r][0] = acc[r][1] = 0.0;
    double big = C64_SCALE;
    asm volatile("" : "+s"(big));
    const uint64_t active = __builtin_amdgcn_read_exec();
    struct Ops { cd2 a[C64_TM / 2], c, base, cut; };
    auto operands = [&](int buf, int k) {
        Ops o;
        o.base = *(const cd2 *)&L.base[buf][k][lane * 2];
        if constexpr (!PLAIN) { o.c = *(const cd2 *)&L.c[buf][k][lane * 2]; o.cut = *(const cd2 *)&L.cut[buf][k][lane * 2]; }
#pragma unroll
        for (int r = 0; r < C64_TM / 2; ++r) o.a[r] = *(const cd2 *)&L.a[buf][k][wave * C64_TM + 2 * r];
        return o;
    };
    auto fold = [&](const Ops &o) {
#pragma unroll
        for (int r = 0; r < C64_TM; r += 2) {
            const double a = o.a[r / 2][0], e = o.a[r / 2][1];
            double t[4];
            if constexpr (PLAIN) {
                // (the discount under the execution mask: mmlike_valu_f64.hip)
                asm volatile("v_mul_f64 %0, %8, %10\n\tv_mul_f64 %1, %8, %11\n\tv_mul_f64 %2, %9, %10\n\tv_mul_f64 %3, %9, %11\n\t"
                             "v_cmpx_gt_f64_e32 vcc, %0, %12\n\tv_mul_f64 %0, %0, %14\n\ts_mov_b64 exec, %16\n\tv_cmpx_gt_f64_e32 vcc, %1, %13\n\tv_mul_f64 %1, %1, %15\n\ts_mov_b64 exec, %16\n\t"
                             "v_cmpx_gt_f64_e32 vcc, %2, %12\n\tv_mul_f64 %2, %2, %14\n\ts_mov_b64 exec, %16\n\tv_cmpx_gt_f64_e32 vcc, %3, %13\n\tv_mul_f64 %3, %3, %15\n\ts_mov_b64 exec, %16\n\t"
                             "v_add_f64 %4, %4, %0\n\tv_add_f64 %5, %5, %1\n\tv_add_f64 %6, %6, %2\n\tv_add_f64 %7, %7, %3"
                             : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1])
                             : "v"(a), "v"(e), "v"(o.base[0]), "v"(o.base[1]), "v"(th[0]), "v"(th[1]), "v"(od[0]), "v"(od[1]), "s"(active) : "vcc");
            } else {
                asm volatile("v_fma_f64 %0, %8, %10, %11 clamp\n\tv_fma_f64 %1, %8, %10, %12 clamp\n\tv_fma_f64 %2, %9, %10, %11 clamp\n\tv_fma_f64 %3, %9, %10, %12 clamp\n\t"
                             "v_fma_f64 %0, %0, -|%13|, %15\n\tv_fma_f64 %1, %1, -|%14|, %16\n\tv_fma_f64 %2, %2, -|%13|, %15\n\tv_fma_f64 %3, %3, -|%14|, %16\n\t"
                             "v_fma_f64 %4, %8, %0, %4\n\tv_fma_f64 %5, %8, %1, %5\n\tv_fma_f64 %6, %9, %2, %6\n\tv_fma_f64 %7, %9, %3, %7"
                             : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "+v"(acc[r][0]), "+v"(acc[r][1]), "+v"(acc[r + 1][0]), "+v"(acc[r + 1][1])
                             : "v"(a), "v"(e), "s"(big), "v"(o.c[0]), "v"(o.c[1]), "v"(o.cut[0]), "v"(o.cut[1]), "v"(o.base[0]), "v"(o.base[1]));
            }
        }
    };
    const int stages = (K + BK - 1) / BK;
    load(K);
    store(0);
    if (PLAIN) __syncthreads();
    else if (refused()) return false;
    for (int t = 0; t < stages; ++t) {
        const int buf = t & 1, k0 = t * BK;
        if (t + 1 < stages) load(K - (t + 1) * BK);
        if (!PLAIN || k0 + BK <= K) {
            // (operands a k ahead, in the registers that the plain way has not)
            Ops o[2];
            if constexpr (!PLAIN) o[0] = operands(buf, 0);
#pragma unroll
            for (int k = 0; k < BK; ++k) {
                if constexpr (PLAIN) o[k & 1] = operands(buf, k);
                else if (k + 1 < BK) o[(k + 1) & 1] = operands(buf, k + 1);
                __builtin_amdgcn_sched_barrier(0);
                fold(o[k & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll 1
            for (int k = k0; k < K; ++k) fold(operands(buf, k - k0));
        }
        if (t + 1 < stages) store(buf ^ 1);
        // (looked at after the first stage, some 64 or 128 k, and twice as many each time, and at the end)
        if (!PLAIN && (t & (t + 1)) == 0 && t >= 7) {
            if (refused()) return false;
        } else __syncthreads();
    }
    if (!PLAIN && refused()) return false;

    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    const int wrow = row0 + wave * C64_TM;
    cd2 old[C64_TM];
    bool last, whole;
    const int col = col_at(l * 2, whole);
    (void)col_at(l * 2 + 1, last);
    whole = whole && last;
#pragma unroll
    for (int r = 0; r < C64_TM; ++r) {
        old[r] = cd2{0, 0};
        if (whole && wrow + r < M) old[r] = *(const cd2_any *)(args.R + (int64_t)(wrow + r) * args.ldr + col);
    }
#pragma unroll
    for (int r = 0; r < C64_TM; ++r) {
        if (wrow + r >= M) break;
        double *const dst_row = args.R + (int64_t)(wrow + r) * args.ldr;
        if (whole) *(cd2_any *)(dst_row + col) = old[r] + cd2{acc[r][0], acc[r][1]};
        else
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int at = col_at(l * 2 + c, own);
                if (own) dst_row[at] += acc[r][c];
            }
    }
    return true;
}

// A tile by critical values, or, if it holds what they do not take, by the task's own operations.
template <int TF, int TRANS, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
mmlike_critical_f64_kernel(const MmlikeArgsF64 args)
{
    extern __shared__ __attribute__((aligned(16))) char critical64_smem[];
    Critical64Lds<NW> &L = *(Critical64Lds<NW> *)critical64_smem;
    const unsigned wave = own_wave();
    if (critical_tile_f64<TF, TRANS, NW, false>(args, threadIdx.x, L)) return;
    unsigned tid;
    const auto &again = opaque_args<MmlikeArgsF64>(wave, tid);
    critical_tile_f64<TF, TRANS, NW, true>(again, tid, L);
}

template <int TF, int TRANS, int NW>
static hipError_t launch_critical_f64(const MmlikeArgsF64 &args, hipStream_t s)
{
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&mmlike_critical_f64_kernel<TF, TRANS, NW>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Critical64Lds<NW>));
    if (granted != hipSuccess) return granted;
    MmlikeArgsF64 b = args;
    const int64_t blocks = xcd_grid(((int64_t)b.M + C64_TM * NW - 1) / (C64_TM * NW), ((int64_t)b.N + C64_COLS - 1) / C64_COLS);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    return launch_row_of_blocks(b, blocks, 64 * NW, [&](unsigned n) {
        hipLaunchKernelGGL((mmlike_critical_f64_kernel<TF, TRANS, NW>), dim3(n), dim3(64 * NW), sizeof(Critical64Lds<NW>), s, b);
    });
}

template <int TF>
hipError_t launch_mmlike_critical_f64(const MmlikeArgsF64 &a, int rows, hipStream_t s)
{
    const int trans = (a.transA ? 1 : 0) | (a.transB ? 2 : 0);
    switch (rows == 64 ? trans : 4 + trans) {
    case 0: return launch_critical_f64<TF, 0, 8>(a, s);
    case 1: return launch_critical_f64<TF, 1, 8>(a, s);
    case 2: return launch_critical_f64<TF, 2, 8>(a, s);
    case 3: return launch_critical_f64<TF, 3, 8>(a, s);
    case 4: return launch_critical_f64<TF, 0, 16>(a, s);
    case 5: return launch_critical_f64<TF, 1, 16>(a, s);
    case 6: return launch_critical_f64<TF, 2, 16>(a, s);
    default: return launch_critical_f64<TF, 3, 16>(a, s);
    }
}

}  // namespace amulet
#endif
