// BOOST in fp32 with its two sums on two units: g = p + max(p - th, 0), and
//
//     sum_k p             on the bf16 matrix cores, from three bf16 pieces per value (pieces.h)
//     sum_k max(p - th, 0) on the vector ALU, two instructions per product:
//         t = clamp(fma(a, b s, -th s));  part += t
//
// where the wide kernel (mmlike_valu_impl.h) takes four.  The clamp modifier costs nothing and bounds to 0 .. 1, so B and
// the thresholds are scaled by s = 2^-52, exactly, and the sums back at the end.  What the two take, in register-only loops
// (clocks of a SIMD per 64 products): fma, fma, max, add 8.4; fma with clamp, add 4.5.  (An instruction with a scalar operand
// or a max may issue beside a plain all-vector one, not beside its like; four waves to a SIMD keep both issue ports fed.)
//
// The rest is the wide kernel's: 32 x 256 outputs per workgroup of eight waves, a lane 4 x 4 of them, A through the
// scalar cache, B staged through LDS 16 k at a time, B's values read a chunk ahead, wave priorities in turns.  To that
// come, per 16 k: the wave's 32 columns of B taken apart into pieces from LDS, the 32 rows of A taken apart by half of the
// threads as they are staged, and six matrix instructions for the 32 x 32 outputs of the wave, all of it
// before the vector loop, whose B values are not live then (in between them, 45 registers too many).  Both sums are
// partial over 64 k: then the matrix cores' goes through LDS into the lanes that own the outputs, the sum of both is added
// to the main accumulators, and what that rounds away starts the next partial sum.  Error against 64 bits, wide kernel / here:
// K = 64 1.5e-7 / 1.0e-7, 512 1.3e-7 / 8.6e-8, 2048 1.2e-7 / 6.0e-8, 4096 1.4e-7 / 5.1e-8 (tile kernels, 4096 x 512 x 8192: 7.7e-8 / 4.9e-8).
//
// us, wide kernel / here: 2048^3 533 / 415 (41 TFLOP/s), 4096^3 4205 / 3240, 8192^2 x 512 2130 / 1680; A transposed 603 / 473, B
// transposed 568 / 441, thres[i][j] 569 / 438.  What bounds it: issue; a matrix instruction
// takes the second issue port for its 32 clocks (0.6 clocks per 64 products), taking B apart once per 32 rows as much
// again, staging and barriers the rest of 6.4 clocks at 2.2 GHz.  DISCOUNT in this manner -- f sum p + (1 - f) sum of the p
// <= th, the predicate a clamp too -- has three vector instructions for its four and was slower, 4297 / 4050 us at 4096^3.
//
// Values it does not take: nonzero |a| or |b| below 2^-36 (products in the subnormal range once scaled, pieces below
// bf16's), triggered parts of 2^51 or more over 64 k (a term at the clamp is one), sums of 2^72 or more, thresholds of
// 0 < |th| < 2^-70, results that are not finite.  A workgroup that finds any of these, at its end, forms its tile again with the wide
// kernel's arithmetic.  The bound on the sums is for the clamp's sake: a partial sum starts at what the fold before it rounded away, less
// than 0.1 for scaled sums below 2^20 (half an ulp of the sum, and of the difference it is found by), and a term at the clamp takes
// it to 0.9 and so beyond the 0.5 it is known by.  (Without it a partial sum could start far below zero, and hide the term.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amulet_internal.h"
#include "pieces.h"

#ifndef AMULET_MMLIKE_BOOST_IMPL_H
#define AMULET_MMLIKE_BOOST_IMPL_H

namespace amulet {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef f4 f4_any __attribute__((aligned(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef f2 f2_any __attribute__((aligned(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) float *sptr_f;

constexpr int BOOST_ROWS = 32, BOOST_COLS = 256, BOOST_BK = 16;
constexpr int BOOST_PITCH = 264;   // floats; rows 4 apart start in different halves of the LDS banks
constexpr float BOOST_SCALE = 0x1p-52f;

struct BoostLds {
    float b[2][BOOST_BK][BOOST_COLS];             // B scaled
    uint32_t a[2][3][BOOST_ROWS][BOOST_BK / 2];   // A's pieces: [piece][row][k pair]
    float s[BOOST_ROWS][BOOST_PITCH];             // the matrix cores' sums of 64 k
};

template <int TF, int TRANS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
mmlike_boost_kernel(const MmlikeArgs args)
{
    constexpr int TM = 4, NW = 8, BK = BOOST_BK, BN = BOOST_COLS, KA = 4;
    constexpr bool transA = (TRANS & 1) != 0, transB = (TRANS & 2) != 0;
    extern __shared__ __attribute__((aligned(16))) char boost_smem[];
    BoostLds &L = *(BoostLds *)boost_smem;
    const int M = args.M, N = args.N;
    int K = args.K;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (M + BOOST_ROWS - 1) / BOOST_ROWS, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    int block = (int)blockIdx.x + args.block_base, ksplit_idx = (int)blockIdx.y;
    const bool tail_part = args.tail_splits > 1 && block >= args.tail_base;
    if (tail_part) {
        const int rel = block - args.tail_base;
        block = args.tail_base + rel % args.tail_blocks;
        ksplit_idx = rel / args.tail_blocks;
    }
    if (!xcd_tile(block, tiles_m, tiles_n, tm, tn)) return;
    const int row0 = tm * BOOST_ROWS + wave * TM, col0 = tn * BN;
    const bool groups = N >= 4;
    auto col_at = [&](int p, bool &own) {
        const int u = col0 + (p & ~3);
        if (groups) {
            const int col = (u < N - 4 ? u : N - 4) + (p & 3);
            own = col >= u;
            return col;
        }
        own = col0 + p < N;
        return own ? col0 + p : N - 1;
    };
    const bool ksplit = gridDim.y > 1 || tail_part;
    int kb = 0;
    if (ksplit) {
        kb = ksplit_idx * args.kchunk;
        K = K - kb < args.kchunk ? K - kb : args.kchunk;
    }
    const float *__restrict__ Ag = args.A + (transA ? (int64_t)kb * args.lda : (int64_t)kb);
    const float *__restrict__ Bg = args.B + (transB ? (int64_t)kb : (int64_t)kb * args.ldb);
    sptr_f As = (sptr_f)Ag;
    auto rowc = [&](int r) { const int row = row0 + r; return row < M ? row : M - 1; };
    const bool rows_full = row0 + TM <= M;
    int64_t arow[transA ? 1 : TM];
    const int arow0 = row0 < M ? row0 : M - 1;
    const int last_valid = (M - arow0 < TM ? M - arow0 : TM) - 1;
    auto trow = [&](int r) { return arow0 + (r < last_valid ? r : last_valid); };
    if constexpr (!transA) {
#pragma unroll
        for (int r = 0; r < TM; ++r) arow[r] = (int64_t)rowc(r) * args.lda;
    } else arow[0] = 0;

    // thresholds, scaled and negated, in vector registers (see the wide kernel); `odd`: outside what the loop takes
    bool odd = false;
    auto held = [&](float t) -> float {
        odd |= __builtin_fabsf(t) < 0x1p-70f && t != 0.0f;
        return -t * BOOST_SCALE;
    };
    float th_col[TF == THRES_COL ? 4 : 1], th_row[TF == THRES_ROW ? TM : 1], th_el[TF == THRES_ELEM ? TM : 1][TF == THRES_ELEM ? 4 : 1];
    float th_const = 0.0f;
    if constexpr (TF == THRES_CONST) { th_const = held(((sptr_f)args.thres)[0]); asm volatile("" : "+v"(th_const)); }
    if constexpr (TF == THRES_ROW) {
#pragma unroll
        for (int r = 0; r < TM; ++r) { th_row[r] = held(((sptr_f)args.thres)[rowc(r)]); asm volatile("" : "+v"(th_row[r])); }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        bool own;
        const int col = col_at(lane * 4 + c, own);
        if constexpr (TF == THRES_COL) th_col[c] = held(args.thres[col]);
        if constexpr (TF == THRES_ELEM)
#pragma unroll
            for (int r = 0; r < TM; ++r) th_el[r][c] = held(args.thres[(int64_t)rowc(r) * args.ldt + col]);
    }
    auto thres = [&](int r, int c) -> float {
        if constexpr (TF == THRES_COL) return th_col[c];
        else if constexpr (TF == THRES_ROW) return th_row[r];
        else if constexpr (TF == THRES_CONST) return th_const;
        else return th_el[r][c];
    };

    float part[TM][4], mainacc[TM][4];
#pragma unroll
    for (int r = 0; r < TM; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) part[r][c] = mainacc[r][c] = 0.0f;
    f16v sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.0f;
    // the least nonzero magnitude staged by this thread (twice its bits, less 1: zeros are the largest), and the largest
    // partial sum of clamped terms, or 2^-21 of a main accumulator
    uint32_t least = 0xffffffffu;
    float most = 0.0f;
    auto see = [&](float x, float y) {
        const uint32_t ux = (__builtin_bit_cast(uint32_t, x) << 1) - 1u, uy = (__builtin_bit_cast(uint32_t, y) << 1) - 1u;
        least = min(least, min(ux, uy));
    };

    // B staging
    constexpr int F4_PER_ROW = BN / 4, LOADS = BK * F4_PER_ROW / 512, ROWS_PER_PASS = 512 / F4_PER_ROW;
    bool own_dummy;
    const int srow = tid / F4_PER_ROW, bcol = col_at((tid % F4_PER_ROW) * 4, own_dummy);
    const float *bsrc = Bg + (int64_t)srow * args.ldb + bcol;
    const int64_t pass_stride = (int64_t)ROWS_PER_PASS * args.ldb, tile_stride = (int64_t)BK * args.ldb;
    constexpr int KPT = BK / 2;
    const int tcol = tid % BN, tk = (tid / BN) * KPT;
    const float *btsrc = Bg + (int64_t)col_at(tcol, own_dummy) * args.ldb + tk;
    f4 stage[LOADS];
    // A pieces: threads 0 .. 255, two k of a row each
    const int prow = transA ? tid & 31 : tid >> 3, pk = (transA ? (tid >> 5) & 7 : tid & 7) * 2;
    const int wrow = tm * BOOST_ROWS + prow < M ? tm * BOOST_ROWS + prow : M - 1;
    const float *psrc = transA ? Ag + (int64_t)pk * args.lda + wrow : Ag + (int64_t)wrow * args.lda + pk;
    f2 pstage = {0.0f, 0.0f};
    auto load_tile = [&](int krows) {
        if (tid < 256) {
            if (krows == BK) {
                if constexpr (transA) { pstage[0] = psrc[0]; pstage[1] = psrc[args.lda]; }
                else pstage = *(const f2_any *)psrc;
            } else {
                pstage[0] = pstage[1] = 0.0f;
                if (pk < krows) pstage[0] = psrc[0];
                if (pk + 1 < krows) pstage[1] = transA ? psrc[args.lda] : psrc[1];
            }
            psrc += transA ? (int64_t)BK * args.lda : BK;
        }
        if (transB) {
            if (krows == BK) {
#pragma unroll
                for (int it = 0; it < LOADS; ++it) stage[it] = *(const f4_any *)(btsrc + 4 * it);
            } else {
                int last = krows - 1;
                asm volatile("" : "+s"(last));
#pragma unroll
                for (int it = 0; it < LOADS; ++it)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int kk = tk + 4 * it + e;
                        stage[it][e] = btsrc[(kk < last ? kk : last) - tk];
                    }
            }
            btsrc += BK;
        } else {
            if (krows == BK && groups) {
#pragma unroll
                for (int it = 0; it < LOADS; ++it) stage[it] = *(const f4_any *)(bsrc + it * pass_stride);
            } else {
                int last = krows - 1;
                asm volatile("" : "+s"(last));
#pragma unroll
                for (int it = 0; it < LOADS; ++it) {
                    const int kk = srow + it * ROWS_PER_PASS;
                    const float *src = bsrc + (int64_t)((kk < last ? kk : last) - srow) * args.ldb;
                    if (groups) stage[it] = *(const f4_any *)src;
                    else
#pragma unroll
                        for (int e = 0; e < 4; ++e) stage[it][e] = src[bcol + e < N ? e : N - 1 - bcol];
                }
            }
            bsrc += tile_stride;
        }
    };
    auto store_tile = [&](int buf) {
        if (tid < 256) {
            uint32_t p0, p1, p2;
            see(pstage[0], pstage[1]);
            take_pieces(pstage[0], pstage[1], p0, p1, p2);
            L.a[buf][0][prow][pk / 2] = p0;
            L.a[buf][1][prow][pk / 2] = p1;
            L.a[buf][2][prow][pk / 2] = p2;
        }
#pragma unroll
        for (int it = 0; it < LOADS; ++it) {
            see(stage[it][0], stage[it][1]);
            see(stage[it][2], stage[it][3]);
            stage[it] *= BOOST_SCALE;
        }
        if (transB) {
#pragma unroll
            for (int it = 0; it < LOADS; ++it)
#pragma unroll
                for (int e = 0; e < 4; ++e) L.b[buf][tk + 4 * it + e][tcol] = stage[it][e];
        } else {
#pragma unroll
            for (int it = 0; it < LOADS; ++it) *(f4 *)&L.b[buf][srow + it * ROWS_PER_PASS][(tid % F4_PER_ROW) * 4] = stage[it];
        }
    };

    const int full_tiles = K / BK, tail = K - full_tiles * BK, n_tiles = full_tiles + (tail ? 1 : 0);
    typedef float av_raw __attribute__((ext_vector_type(KA)));
    typedef av_raw av_t __attribute__((aligned(4)));
    typedef const __attribute__((address_space(4))) av_t *sptr_av;
    av_t a_next[TM];
    auto a_of = [](const av_t (&v)[TM], int r, int kk) -> float { return transA ? v[kk][r] : v[r][kk]; };
    auto fetch_a = [&](int kt, int rel) {
        const int kn = kt + rel;
        if constexpr (!transA) {
            uint32_t relb = (uint32_t)rel * 4u;
            asm volatile("" : "+s"(relb));
            typedef const __attribute__((address_space(4))) char *sptr_c;
#pragma unroll
            for (int r = 0; r < TM; ++r) a_next[r] = *(sptr_av)((sptr_c)(As + (arow[r] + kt)) + relb);
        } else if (rows_full) {
#pragma unroll
            for (int kk = 0; kk < KA; ++kk) a_next[kk] = *(sptr_av)(As + (int64_t)(kn + kk) * args.lda + arow0);
        } else {
#pragma unroll
            for (int kk = 0; kk < KA; ++kk)
#pragma unroll
                for (int r = 0; r < TM; ++r) a_next[kk][r] = As[(int64_t)(kn + kk) * args.lda + trow(r)];
        }
    };
    load_tile(full_tiles > 0 ? BK : tail);
    store_tile(0);
    if (full_tiles > 0) fetch_a(0, 0);
    __syncthreads();

    // the tile's products on the matrix cores: the wave's 32 columns of B
    auto matrix_part = [&](int buf) {
        float raw[8];
        u4 bp[3], ap[3];
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[i] = L.b[buf][8 * lh + i][wave * 32 + li];
#pragma unroll
        for (int q = 0; q < 3; ++q) ap[q] = *(const u4 *)&L.a[buf][q][li][lh * 4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t p0, p1, p2;
            take_pieces(raw[2 * i], raw[2 * i + 1], p0, p1, p2);
            bp[0][i] = p0; bp[1][i] = p1; bp[2][i] = p2;
        }
        constexpr int PA[6] = {2, 1, 1, 0, 0, 0}, PB[6] = {0, 0, 1, 1, 0, 2};
#pragma unroll
        for (int i = 0; i < 6; ++i)
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, ap[PA[i]]), __builtin_bit_cast(bf8, bp[PB[i]]), sum, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto dump = [&]() {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            L.s[8 * (v >> 2) + 4 * lh + (v & 3)][wave * 32 + li] = sum[v];
            sum[v] = 0.0f;
        }
    };
    auto fold = [&]() {
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const f4 s4 = *(const f4 *)&L.s[wave * TM + r][lane * 4];
            float sums = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // (what the addition rounds away starts the next partial sum)
                const float v = part[r][c] + s4[c], m = mainacc[r][c] + v;
                most = __builtin_fmaxf(most, part[r][c]);
                sums = __builtin_fmaxf(sums, __builtin_fabsf(m));
                part[r][c] = v - (m - mainacc[r][c]);
                mainacc[r][c] = m;
            }
            most = __builtin_fmaxf(most, sums * 0x1p-21f);
        }
    };
    auto term = [&](float a, float b, int r, int c) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(a, b, thres(r, c)), 0.0f, 1.0f); };
    // a chunk of 4 k: the fma of product i, then the addition of product i - 1 (one scalar operand to two instructions)
    auto compute_chunk = [&](const av_t (&a)[TM], const f4 (&b)[KA]) {
        constexpr int NP = KA * TM * 4;
        float t[NP];
#pragma unroll
        for (int i = 0; i <= NP; ++i) {
            if (i < NP) t[i] = term(a_of(a, i / 4 % TM, i / 16), b[i / 16][i % 4], i / 4 % TM, i % 4);
            __builtin_amdgcn_sched_barrier(0);
            if (i >= 1) part[(i - 1) / 4 % TM][(i - 1) % 4] += t[i - 1];
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const int prio_phase = block >> 8;
    for (int t = 0; t < n_tiles; ++t) {
        const int buf = t & 1, k0 = t * BK;
        switch ((t + prio_phase) & 3) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
        }
        if (t > 0 && (t & 3) == 0) fold();
        if (t + 1 < n_tiles) load_tile(t + 1 < full_tiles ? BK : tail);
        const float *bs = &L.b[buf][0][lane * 4];
        matrix_part(buf);
        if (t < full_tiles) {
            if constexpr (!transA) {
                // the B values of a chunk are read while the chunk before it computes
                f4 bq[2][KA];
#pragma unroll
                for (int kk = 0; kk < KA; ++kk) bq[0][kk] = *(const f4 *)(bs + kk * BN);
#pragma unroll
                for (int c = 0; c < BK / KA; ++c) {
                    const int kc = c * KA;
                    av_t a[TM];
#pragma unroll
                    for (int r = 0; r < TM; ++r) a[r] = a_next[r];
                    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this chunk's B and A values have landed
                    __builtin_amdgcn_sched_barrier(0);
                    if (c + 1 < BK / KA) {
#pragma unroll
                        for (int kk = 0; kk < KA; ++kk) bq[(c + 1) & 1][kk] = *(const f4 *)(bs + (kc + KA + kk) * BN);
                        fetch_a(k0, kc + KA);
                    } else fetch_a(k0, k0 + BK + KA <= K ? BK : BK - KA);   // (past the last full chunk: this one again)
                    __builtin_amdgcn_sched_barrier(0);
                    compute_chunk(a, bq[c & 1]);
                }
            } else {
                // (unrolled, a transposed A's values of all chunks are in scalar registers at once: 80 too many)
#pragma unroll 1
                for (int kc = 0; kc < BK; kc += KA) {
                    f4 b[KA];
#pragma unroll
                    for (int kk = 0; kk < KA; ++kk) b[kk] = *(const f4 *)(bs + (kc + kk) * BN);
                    av_t a[TM];
#pragma unroll
                    for (int r = 0; r < TM; ++r) a[r] = a_next[r];
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    __builtin_amdgcn_sched_barrier(0);
                    fetch_a(k0, k0 + kc + 2 * KA <= K ? kc + KA : kc);
                    __builtin_amdgcn_sched_barrier(0);
                    compute_chunk(a, b);
                }
            }
        } else {
            for (int kk = 0; kk < tail; ++kk) {
                const f4 b = *(const f4 *)(bs + kk * BN);
#pragma unroll
                for (int r = 0; r < TM; ++r) {
                    const float a1 = transA ? As[(int64_t)(k0 + kk) * args.lda + trow(r)] : As[arow[transA ? 0 : r] + k0 + kk];
#pragma unroll
                    for (int c = 0; c < 4; ++c) part[r][c] += term(a1, b[c], r, c);
                }
            }
        }
        // (a last tile that began with a fold: every wave has to have read its sums before they are overwritten)
        if (t + 1 == n_tiles && t > 0 && (t & 3) == 0) __syncthreads();
        if ((t & 3) == 3 || t + 1 == n_tiles) dump();
        if (t + 1 < n_tiles) store_tile(buf ^ 1);
        __syncthreads();
    }
    fold();
    // (opaque from here on, or what follows has its columns computed before the K loop and held through it)
    int l = lane;
    asm volatile("" : "+v"(l));
    bool again = odd || least < (0x2dc00000u << 1) - 1u || !(most < 0.5f);   // (2^-36)
#pragma unroll
    for (int r = 0; r < TM; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            mainacc[r][c] *= 1.0f / BOOST_SCALE;
            again |= !(__builtin_fabsf(mainacc[r][c]) <= 3.402823466e+38f);
        }
    if (__syncthreads_or(again)) {
        // the wide kernel's arithmetic, from global memory
        float th[TM][4];
        int cols[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            bool own;
            cols[c] = col_at(l * 4 + c, own);
#pragma unroll
            for (int r = 0; r < TM; ++r) {
                th[r][c] = args.thres[TF == THRES_COL ? cols[c] : TF == THRES_ROW ? rowc(r) : TF == THRES_CONST ? 0 : (int64_t)rowc(r) * args.ldt + cols[c]];
                mainacc[r][c] = part[r][c] = 0.0f;
            }
        }
#pragma unroll 1
        for (int k = 0; k < K; ++k) {
            float b[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = transB ? Bg[(int64_t)cols[c] * args.ldb + k] : Bg[(int64_t)k * args.ldb + cols[c]];
#pragma unroll
            for (int r = 0; r < TM; ++r) {
                const float a = transA ? As[(int64_t)k * args.lda + trow(r)] : As[arow[transA ? 0 : r] + k];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float d = __builtin_fmaf(a, b[c], -th[r][c]);
                    part[r][c] = __builtin_fmaf(a, b[c], part[r][c]) + __builtin_fmaxf(d, 0.0f);
                }
            }
            if ((k & 63) == 63 || k + 1 == K)
#pragma unroll
                for (int r = 0; r < TM; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) { mainacc[r][c] += part[r][c]; part[r][c] = 0.0f; }
        }
    }

    if (ksplit) {
        float *const x = &L.b[0][0][0] + wave * 256;
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            if (row0 + r >= M) break;
            float *const dst_row = args.R + (int64_t)(row0 + r) * args.ldr;
            *(f4 *)(x + l * 4) = f4{mainacc[r][0], mainacc[r][1], mainacc[r][2], mainacc[r][3]};
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bool own;
                const int col = col_at(c * 64 + l, own);
                if (own) unsafeAtomicAdd(dst_row + col, x[c * 64 + l]);
            }
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
    f4 old[TM];
    bool whole, last;
    const int col = col_at(l * 4, whole);
    (void)col_at(l * 4 + 3, last);
    whole = whole && last;
#pragma unroll
    for (int r = 0; r < TM; ++r) {
        old[r] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        if (whole && row0 + r < M) old[r] = *(const f4_any *)(args.R + (int64_t)(row0 + r) * args.ldr + col);
    }
#pragma unroll
    for (int r = 0; r < TM; ++r) {
        if (row0 + r >= M) break;
        float *dst_row = args.R + (int64_t)(row0 + r) * args.ldr;
        f4 o = old[r];
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] += mainacc[r][c];
        if (whole) *(f4_any *)(dst_row + col) = o;
        else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bool own;
                const int at = col_at(l * 4 + c, own);
                if (own) dst_row[at] += o[c];
            }
        }
    }
}

template <int TF, int TRANS>
static hipError_t launch_boost(MmlikeArgs &b, int64_t blocks, int splits, hipStream_t s)
{
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&mmlike_boost_kernel<TF, TRANS>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(BoostLds));
    if (granted != hipSuccess) return granted;
    return launch_row_of_blocks(b, blocks, 512, [&](unsigned n) {
        hipLaunchKernelGGL((mmlike_boost_kernel<TF, TRANS>), dim3(n, (unsigned)splits), dim3(512), sizeof(BoostLds), s, b);
    });
}

template <int TF>
hipError_t launch_mmlike_boost(const MmlikeArgs &args, hipStream_t s)
{
    MmlikeArgs b = args;
    const int64_t tiles_m = ((int64_t)b.M + BOOST_ROWS - 1) / BOOST_ROWS, tiles_n = ((int64_t)b.N + BOOST_COLS - 1) / BOOST_COLS;
    int64_t blocks = xcd_grid(tiles_m, tiles_n);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // K in the parts of the wide kernel: every tile's where tiles are few, else the last round's
    const int64_t chunk = wide_k_range(tiles_m * tiles_n * 8, b.K);
    b.kchunk = (int)chunk;
    const int splits = (int)((b.K + chunk - 1) / chunk);
    b.tail_base = 0; b.tail_blocks = 0; b.tail_splits = 1;
    TailSplit t;
    if (splits == 1 && choose_tail_split(tiles_m * tiles_n, blocks, (int64_t)compute_units() * 2, b.K, 64, t)) {
        b.tail_base = (int)t.base;
        b.tail_blocks = (int)t.blocks;
        b.tail_splits = t.splits;
        b.kchunk = t.chunk;
        blocks = t.grid;
    }
    switch ((b.transA ? 1 : 0) | (b.transB ? 2 : 0)) {
    case 0: return launch_boost<TF, 0>(b, blocks, splits, s);
    case 1: return launch_boost<TF, 1>(b, blocks, splits, s);
    case 2: return launch_boost<TF, 2>(b, blocks, splits, s);
    default: return launch_boost<TF, 3>(b, blocks, splits, s);
    }
}

}  // namespace amulet
#endif
