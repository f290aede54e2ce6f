// fp32 VALU tile kernels for the matrix-multiplication-like tasks whose g acts
// on each product before the k-sum (paper Fig. 1, Fig. 2, Query 1-3): these
// cannot run on the matrix cores, so the inner kernel is a per-lane register
// micro-tile on the vector ALU, the CDNA form of the paper's register-blocked
// inner kernel (Sec. 3, Fig. "12x16 inner kernel"; Sec. 4.3.3 for the version
// with g inside the kk loop).
//
// Mapping (one workgroup = NW waves, one R tile of NW*TM rows x 256*NG columns):
//   * a lane owns 4*NG columns: column groups g*256 + lane*4 .. +3.  thres[j]
//     and the per-column factor derived from dis[j] live in registers for the
//     whole K loop (the paper reloads them every kk and budgets registers for
//     them, Sec. 4.3.2).
//   * a wave owns TM rows, the same for all its lanes, so A[i][k] is wave
//     uniform: it is fetched through the scalar data cache into SGPRs and used
//     directly as the scalar operand of the multiply.  A never touches LDS or
//     vector registers.
//   * the BK x (256*NG) tile of B is staged global -> registers -> LDS, double
//     buffered, one barrier per tile; a lane reads its own 16-byte column groups
//     back with conflict-free ds_read_b128.
//   * the k-sum is two-level: a partial accumulator over FLUSH_K products,
//     folded into the main accumulator after that many, which keeps fp32
//     round-off of long same-sign sums (K = 8192 retail data) far inside the
//     1e-5 budget.
//   * the K remainder is computed by a k-by-k tail loop, never by zero padding:
//     g(0) is not 0 in general (BOOST with thres < 0, COUNT_GT with thres < 0).
//
// Per product the discount task costs 4 VALU lane-operations (multiply rounded
// to fp32, compare, select of the factor, fused multiply-add), the paper's
// sequence "mul, gtcmp, mul, masksub, add" (Sec. 4.3.1) minus one.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "amulet_internal.h"
#include "boost_pieces.h"
#include "count_rounding.h"

#ifndef AMULET_MMLIKE_VALU_IMPL_H
#define AMULET_MMLIKE_VALU_IMPL_H

namespace amulet {

// k-extent of one partial sum of the two-level fp32 accumulation
constexpr int FLUSH_K = 64;

typedef float f4 __attribute__((ext_vector_type(4)));
// the same four floats at any float address: still one 16-byte access (global accesses take
// any address on this target), used where rows are not 16-byte aligned
typedef f4 f4_any __attribute__((aligned(4)));
typedef const __attribute__((address_space(4))) float *sptr_f;      // read through the scalar cache

// partial and main accumulators: the count task keeps a product's predicate bit, one bit per
// product of a partial sum, and counts them when they are folded in
template <int TASK> struct AccT { typedef float type, main_type; };
template <> struct AccT<TASK_COUNT_GT> { typedef uint32_t type; typedef int main_type; };
// k of one partial sum: 64, or the 32 bits of the count task's partial
template <int TASK> constexpr int partial_k() { return TASK == TASK_COUNT_GT ? 32 : FLUSH_K; }

// Four products of one A value with a lane's group of four B values, folded
// into the (partial) accumulators.  The multiply is a separately rounded fp32
// operation wherever a comparison depends on it.  The four compares are issued
// back to back before the four selects, so each select is at least three
// instructions behind the compare whose mask it reads (the distance gfx950
// wants between a VALU write of a lane mask and its VALU read).
template <int TASK>
__device__ __forceinline__ void fold4(float a, f4 b, const float *th, const float *q,
                                      typename AccT<TASK>::type *acc)
{
    if constexpr (TASK == TASK_IDENTITY) {
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = __builtin_fmaf(a, b[c], acc[c]);
    } else if constexpr (TASK == TASK_DISCOUNT) {
        float p[4], s[4];
        bool m[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = a * b[c];          // one RN multiply (contraction is off)
#pragma unroll
        for (int c = 0; c < 4; ++c) m[c] = p[c] > th[c];
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = m[c] ? q[c] : 1.0f;  // q = 1 - dis[j]
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = __builtin_fmaf(p[c], s[c], acc[c]);
    } else if constexpr (TASK == TASK_BOOST) {
        // p + (p > th)(p - th) = p + max(p - th, 0) is continuous in p, so the
        // unrounded product inside the fused operations is within tolerance.
        // One product at a time, fenced: fma, fma, max, add.  Three of the four read a scalar
        // register or an inline constant, and long runs of such instructions issue slower than
        // the same instructions interleaved with the all-vector add (register-only loops: 9.1-9.7
        // clocks per 64 products in groups of four, 8.4 one at a time; the kernel 30.3 -> 32.3
        // TFLOP/s at 8192^3).  Left alone the scheduler builds pairs and runs of ten.
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float d = __builtin_fmaf(a, b[c], -th[c]);
            acc[c] = __builtin_fmaf(a, b[c], acc[c]);
            d = __builtin_fmaxf(d, 0.0f);
            acc[c] += d;
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // The count needs no lane mask: p > th exactly when th - p is negative (a difference of
        // two floats is zero only when they are equal, subnormal results included, and x - x is
        // +0), so the sign bit of the rounded difference is the predicate bit.  The one
        // exception, -0 - (+0) = -0, is excluded by the caller: it never passes a threshold of -0.
        // v_alignbit_b32 shifts that bit into the partial in one instruction -- multiply, subtract,
        // alignbit, and one bit count per 32 products -- where shifting it down and adding it
        // took one and a half (register-only loops, 4 waves per SIMD: 8.3 against 6.5 clocks per 64
        // products; compare and add with carry 9.9).  The kernel at 4096^3: 38.9 -> 42.7 TFLOP/s.
        // (Thresholds per output, and those that counting by rounding leaves to it.)
        float p[4], d[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = a * b[c];          // one RN multiply (contraction is off)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) d[c] = th[c] - p[c];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_alignbit(acc[c], __builtin_bit_cast(uint32_t, d[c]), 31);
    }
}

// ALDS: the workgroup's rows of A go through LDS too (vector loads a whole tile ahead, then
// broadcast reads), instead of through the scalar cache chunk by chunk.  Slightly more
// registers and LDS traffic; used when the row pitch of A collides (amulet_pitch_collides):
// the scalar path fetches each 128-byte line of A in eight pieces, and when the lines of a
// workgroup's 32 rows all fall into the same L2 sets they are evicted between the pieces.
// PIPE (discount task, 4 x 4 micro-tile): a chunk runs as one software pipeline instead of k by k
// (see the chunk loop); the launcher says when.
template <int TASK, int TF, int TRANS, int TM, int NG, int NW, int BK, int KA, bool ALDS, bool PIPE, bool BPRE, bool PIECES, bool ROUNDED, bool ZERO, typename Args>
__device__ __forceinline__ bool valu_tile(const Args &args, const unsigned tid, float (&Bs)[2][BK][256 * NG],
                                          float (&Asl)[ALDS ? 2 : 1][ALDS ? NW * TM : 1][ALDS ? BK + 4 : 4])
{
    constexpr bool SECOND = !PIECES && !ROUNDED;
    auto done = [](bool whole) { return whole; };
#include "mmlike_valu_tile.inc"
}

template <int TASK, int TF, int TRANS, int TM, int NG, int NW, int BK, int KA, bool ALDS, bool PIPE = false, bool BPRE = false>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(TM * NG == 4 ? 4 : 1)))
mmlike_valu_kernel(const MmlikeArgs args)
{
    __shared__ __attribute__((aligned(16))) float Bs[2][BK][256 * NG];
    __shared__ __attribute__((aligned(16))) float Asl[ALDS ? 2 : 1][ALDS ? NW * TM : 1][ALDS ? BK + 4 : 4];
    if constexpr (TASK == TASK_COUNT_GT && TF != THRES_ELEM && TM == 4 && NG == 1) {
        // by rounding; where every threshold of the tile is 0, by rounding too; or all of the tile again by comparison
        const unsigned wave = own_wave();
        if (valu_tile<TASK, TF, TRANS, TM, NG, NW, BK, KA, ALDS, PIPE, BPRE, false, true, false>(args, threadIdx.x, Bs, Asl)) return;
        unsigned tid;
        const auto &again = opaque_args<MmlikeArgs>(wave, tid);
        if (valu_tile<TASK, TF, TRANS, TM, NG, NW, BK, KA, ALDS, PIPE, BPRE, false, true, true>(again, tid, Bs, Asl)) return;
        const auto &last = opaque_args<MmlikeArgs>(wave, tid);
        valu_tile<TASK, TF, TRANS, TM, NG, NW, BK, KA, ALDS, PIPE, BPRE, false, false, false>(last, tid, Bs, Asl);
    } else {
        constexpr bool PIECES = false, ROUNDED = false, ZERO = false, SECOND = false;
        const unsigned tid = threadIdx.x;
        auto done = [](bool) {};
#include "mmlike_valu_tile.inc"
    }
}

template <int TASK, int TF, int TM, int NG, int NW, int BK, int KA>
static hipError_t launch_one(const MmlikeArgs &a, hipStream_t s)
{
    const int64_t tiles_m = (a.M + NW * TM - 1) / (NW * TM);
    const int64_t tiles_n = (a.N + 256 * NG - 1) / (256 * NG);
    const int64_t wgs = xcd_grid(tiles_m, tiles_n);
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    // few tiles: K over several workgroups (wide_k_range in amulet_internal.h)
    MmlikeArgs b = a;
    int splits = 1;
    b.kchunk = a.K;
    const int64_t waves = tiles_m * tiles_n * NW;
    if (a.force_splits > 1) {
        // a k-axis point of the shape grid: every tile's K in (up to) force_splits parts of whole
        // partial-sum periods; nothing to split in the deterministic mode or when K is short
        if (k_split_allowed() && a.K >= 128) {
            int64_t want = a.force_splits;
            if (want > a.K / 64) want = a.K / 64;
            const int64_t chunk = ((a.K + want - 1) / want + 63) / 64 * 64;
            b.kchunk = (int)chunk;
            splits = (int)((a.K + chunk - 1) / chunk);
        }
    } else {
        const int64_t chunk = wide_k_range(waves, a.K);
        b.kchunk = (int)chunk;
        splits = (int)((a.K + chunk - 1) / chunk);
    }
    b.tail_base = 0; b.tail_blocks = 0; b.tail_splits = 1;
    // Discount task.  With 16-deep staging and A on the scalar path the kernel runs a chunk as one
    // compare / multiply / FMA / select pipeline whose B values were read from LDS a chunk ahead,
    // at every size (8192^3 31.9 -> 34.2 TFLOP/s, 4096^3 32.8 -> 33.9, 16384 x 2048 x 8192 33.1 ->
    // 34.0: the pipeline alone was no faster at 8192^3, the earlier reads alone gave +1.5 %).
    // The other discount instantiations (8-deep staging, A through LDS) keep the pipeline without
    // the earlier reads up to 4096 workgroups, where it measured 2-4 % faster, and the k-by-k form
    // above that.
    const bool pipe = TASK == TASK_DISCOUNT && TM == 4 && NG == 1 && wgs <= 4096;
    // Rows of a row-major A whose pitch collides in the memory system go through LDS; at other
    // pitches the scalar path is as fast or faster for every task (measured at 2048^3 ... 8192^3,
    // A through LDS against A through the scalar cache: discount 30.4-31.0 against 31.3-31.9
    // TFLOP/s, count 36.4-37.2 against 36.9-40.4, boost within +-4 % either way).
    const bool a_through_lds = !a.transA && !a.transB && pitch_collides(a.lda, 4);
    // The count spends the least arithmetic on a stage of B (three instructions per product) and gains by
    // fewer barriers: 32 k a stage, two workgroups' 128 KiB of LDS to a unit (with the fences in fold4, 43.0 -> 44.4
    // TFLOP/s at 4096^3, with A transposed 32.2 -> 38.8; boost is level with it, 32.6 / 32.7).
    constexpr int DEEP = TASK == TASK_COUNT_GT && TM == 4 && NG == 1 && NW == 8 && BK == 16 ? 32 : BK;
    // Discount with A transposed, whose scalar loads of four rows at a time are a longer chain per stage: as deep (us, 16 k /
    // 32: 8192^3 34 900 / 33 930, 4096^3 4382 / 4190, 2048^3 556 / 531, 5501 x 2560 x 833 801 / 768, 2048^2 x 128 44.2 / 40.4, both operands transposed
    // 4427 / 4268 at 4096^3); level with A row-major (4164 / 4159), where 3 registers too many spill in some forms, as with both
    // transposed and a threshold per output.
    constexpr int DEEP_AT = TASK == TASK_DISCOUNT && TM == 4 && NG == 1 && NW == 8 && BK == 16 ? 32 : DEEP;
    constexpr bool DPIPE = TASK == TASK_DISCOUNT && TM == 4 && NG == 1 && BK == 16;
    constexpr bool BAHEAD = TASK != TASK_IDENTITY && TM == 4 && NG == 1 && BK == 16;   // B values a chunk ahead
    auto launch = [&](int64_t n_blocks, int n_splits) -> hipError_t {
        return launch_row_of_blocks(b, n_blocks, 64 * NW, [&](unsigned n) {
            const dim3 grid(n, (unsigned)n_splits), block(64 * NW);
            switch ((a.transA ? 1 : 0) | (a.transB ? 2 : 0)) {
            case 0:
                if constexpr (TASK == TASK_DISCOUNT && TM == 4 && NG == 1 && BK == 16) {
                    // the chunk-wide pipeline fed with B values read a chunk ahead: at every size
                    if (!a_through_lds) {
                        hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, BK, KA, false, true, true>), grid, block, 0, s, b);
                        break;
                    }
                }
                if constexpr ((TASK == TASK_BOOST || TASK == TASK_COUNT_GT) && TM == 4 && NG == 1 && BK == 16) {
                    // B values read a chunk ahead (no chunk pipeline: these tasks have no lane mask
                    // to keep at a distance): boost +0.5-1.5 %, count +1 % (42.7 -> 43.0 TFLOP/s at 4096^3)
                    if (!a_through_lds) {
                        hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, DEEP, KA, false, false, true>), grid, block, 0, s, b);
                        break;
                    }
                }
                if constexpr (TASK == TASK_DISCOUNT && TM == 4 && NG == 1) {
                    if (pipe) {
                        if (a_through_lds)
                            hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, BK, KA, true, true>), grid, block, 0, s, b);
                        else
                            hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, BK, KA, false, true>), grid, block, 0, s, b);
                        break;
                    }
                }
                if constexpr (TM == 4 && NG == 1) {
                    if (a_through_lds) {
                        hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, BK, KA, true>), grid, block, 0, s, b);
                        break;
                    }
                }
                hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 0, TM, NG, NW, BK, KA, false>), grid, block, 0, s, b);
                break;
            // (transposed layouts: the discount task's pipelined form; with B a chunk ahead where A
            // is row-major -- with a transposed A the unrolled tile keeps the A values of all its
            // chunks in scalar registers at once and spills 80-130 of them)
            case 1: hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 1, TM, NG, NW, DEEP_AT, KA, false, DPIPE, false>), grid, block, 0, s, b); break;
            case 2: hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 2, TM, NG, NW, DEEP, KA, false, DPIPE, BAHEAD>), grid, block, 0, s, b); break;
            default: hipLaunchKernelGGL((mmlike_valu_kernel<TASK, TF, 3, TM, NG, NW, TF == THRES_ELEM ? DEEP : DEEP_AT, KA, false, DPIPE, false>), grid, block, 0, s, b); break;
            }
        });
    };
    // a last round of workgroups that would leave most of the chip idle: its tiles are launched
    // once per k range instead (choose_tail_split in amulet_internal.h)
    TailSplit t;
    if (splits == 1 && a.force_splits <= 1 && choose_tail_split(tiles_m * tiles_n, wgs, (int64_t)compute_units() * (16 / NW), a.K, 64, t)) {
        b.tail_base = (int)t.base;
        b.tail_blocks = (int)t.blocks;
        b.tail_splits = t.splits;
        b.kchunk = t.chunk;
        return launch(t.grid, 1);
    }
    return launch(wgs, splits);
}

// Shape id = k-axis index * VALU_TILES + tile index (see amulet_internal.h).
template <int TASK, int TF>
hipError_t launch_mmlike_valu_task(int shape, const MmlikeArgs &args, hipStream_t s)
{
    if (shape < 0 || shape >= VALU_SHAPE_COUNT) return hipErrorInvalidValue;
    MmlikeArgs a = args;
    a.force_splits = kValuShapes[shape].splits;
    const int tile = shape % VALU_TILES;
    if (kValuShapes[shape].BK == 8) {
        switch (tile) {
        case 0: return launch_one<TASK, TF, 4, 1, 4, 8, 4>(a, s);
        case 1: return launch_one<TASK, TF, 4, 1, 8, 8, 4>(a, s);
        case 2: return launch_one<TASK, TF, 8, 1, 8, 8, 4>(a, s);
        default: return launch_one<TASK, TF, 4, 2, 8, 8, 4>(a, s);
        }
    }
    switch (tile) {
    case 0: return launch_one<TASK, TF, 4, 1, 4, 16, 4>(a, s);
    case 1: return launch_one<TASK, TF, 4, 1, 8, 16, 4>(a, s);
    case 2: return launch_one<TASK, TF, 8, 1, 8, 16, 4>(a, s);
    default: return launch_one<TASK, TF, 4, 2, 8, 16, 4>(a, s);
    }
}

}  // namespace amulet
#endif
