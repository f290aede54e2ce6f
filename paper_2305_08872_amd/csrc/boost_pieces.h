// BOOST in fp32 with its two sums on two units: g = p + max(p - th, 0), and
//
//     sum_k p             on the bf16 matrix cores, from three bf16 pieces per value (pieces.h)
//     sum_k max(p - th, 0) on the vector ALU, two instructions per product:
//         t = clamp(fma(a, b s, -th s));  part += t
//
// where the wide kernel's own arithmetic (mmlike_valu_impl.h, fold4) takes four.  The clamp modifier costs nothing and bounds to
// 0 .. 1, so B and the thresholds are scaled by s = 2^-52, exactly, and the sums back at the end.  What the two take, in
// register-only loops (clocks of a SIMD per 64 products): fma, fma, max, add 8.4; fma with clamp, add 4.5.  (An instruction with
// a scalar operand or a max may issue beside a plain all-vector one, not beside its like; four waves to a SIMD keep both issue
// ports fed.)
//
// The rest is the wide kernel, 32 x 256 outputs per workgroup of eight waves.  To that
// come, per 16 k: the wave's 32 columns of B taken apart into pieces from LDS, the 32 rows of A taken apart by half of the
// threads as they are staged, and six matrix instructions for the 32 x 32 outputs of the wave, all of it
// before the vector loop, whose B values are not live then (in between them, 45 registers too many).  Both sums are
// partial over 64 k: then the matrix cores' goes through LDS into the lanes that own the outputs, the sum of both is added
// to the main accumulators, and what that rounds away starts the next partial sum.  Error against 64 bits, wide kernel / here:
// K = 64 1.5e-7 / 9.5e-8, 512 1.2e-7 / 7.9e-8, 2048 1.2e-7 / 5.7e-8 (tile kernels, 4096 x 512 x 8192: 7.7e-8 / 4.9e-8); of a product
// that stands alone in its sum, on average 2.2e-8 / 2.7e-8 and at most 6.0e-8 / 1.5e-7, with its triggered part 2.4e-8 / 3.1e-8 and 7.9e-8 / 1.5e-7.
//
// us, wide kernel / here, operands that change from call to call: 2048^3 545 / 422 (40.7 TFLOP/s), 4096^3 4350 / 3370, 8192^2 x 512 2190 /
// 1745; A transposed 582 / 484, B transposed 552 / 434, thres[i][j] 549 / 434.  What bounds it: issue; a matrix instruction
// takes the second issue port for its 32 clocks (0.6 clocks per 64 products), taking B apart once per 32 rows as much
// again, staging and barriers the rest of 6.4 clocks at 2.2 GHz.  DISCOUNT in this manner -- f sum p + (1 - f) sum of the p
// <= th, the predicate a clamp too -- has three vector instructions for its four and was slower, 4297 / 4050 us at 4096^3.
//
// Values it does not take: nonzero |a| or |b| below 2^-36 (products in the subnormal range once scaled, pieces below
// bf16's), triggered parts of 2^51 or more over 64 k (a term at the clamp is one), sums that round by as much (2^75 and more),
// thresholds of 0 < |th| < 2^-70, results that are not finite.  A workgroup that finds any of these forms its tile again by the
// wide kernel's own arithmetic; it looks at the end, and, for all but the last kind, after 64 k, 128 k, 256 k ..., so that operands
// that are full of them cost little more than that arithmetic alone.  (The bound on what sums round by is for the clamp's sake:
// with it a partial sum starts above -1/2, scaled, and a term at the clamp takes it to the 1/2 it is known by; without it a start
// far below zero hides the term.)  2048^3, us, none of these / one, early in K / one, late, or an infinity / all values / the wide
// kernel: 414 / 470 / 680 / 557 / 537; A transposed 480 / 538 / 849 / 595 / 575, B transposed 419 / 492 / 683 / 561 / 543; one, late,
// in every 32 rows 965.  (k by k from global memory, as this once did: 414 / 1307 / 1309 / 2180, B transposed 5490.)
#ifndef AMULET_BOOST_PIECES_H
#define AMULET_BOOST_PIECES_H
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pieces.h"

namespace amulet {

constexpr int BOOST_ROWS = 32, BOOST_COLS = 256, BOOST_BK = 16;
constexpr int BOOST_PITCH = 264;   // floats; rows 4 apart start in different halves of the LDS banks
constexpr float BOOST_SCALE = 0x1p-52f;

struct BoostLds {
    float b[2][BOOST_BK][BOOST_COLS];             // B scaled
    uint32_t a[2][3][BOOST_ROWS][BOOST_BK / 2];   // A's pieces: [piece][row][k pair]
    float s[BOOST_ROWS][BOOST_PITCH];             // the matrix cores' sums of 64 k
    uint32_t refused[8];                          // by wave
};

// a triggered term, scaled (b and the threshold carry the scale)
__device__ __forceinline__ float boost_term(float a, float b, float th) { return __builtin_amdgcn_fmed3f(__builtin_fmaf(a, b, -th), 0.0f, 1.0f); }

template <bool transA>
struct BoostPieces {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef f2 f2_any __attribute__((aligned(4)));
    typedef float f4v __attribute__((ext_vector_type(4)));
    typedef float f16v __attribute__((ext_vector_type(16)));
    typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    static constexpr int TM = 4, BK = BOOST_BK;

    BoostLds &L;
    int tid, lane, wave, prow, pk;
    int64_t lda;
    const float *psrc;            // this thread's two values of A in the next stage
    f2 pstage = {0.0f, 0.0f};
    f16v sum;
    // the least nonzero magnitude staged by this thread (twice its bits, less 1: zeros are the largest), and the largest
    // partial sum of clamped terms or start of one; `odd`: a threshold outside what the loop takes
    uint32_t least = 0xffffffffu;
    float most = 0.0f;
    bool odd = false;

    // A pieces: threads 0 .. 255, two k of a row each
    __device__ __forceinline__ BoostPieces(BoostLds &lds, const float *A, int64_t pitch, int first_row, int M, int thread, int wave_) : L(lds), tid(thread), lane(thread & 63), wave(wave_), lda(pitch)
    {
        prow = transA ? tid & 31 : tid >> 3;
        pk = (transA ? (tid >> 5) & 7 : tid & 7) * 2;
        const int row = first_row + prow < M ? first_row + prow : M - 1;
        psrc = transA ? A + (int64_t)pk * lda + row : A + (int64_t)row * lda + pk;
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = 0.0f;
    }
    __device__ __forceinline__ float threshold(float t)
    {
        odd |= __builtin_fabsf(t) < 0x1p-70f && t != 0.0f;
        return t * BOOST_SCALE;
    }
    __device__ __forceinline__ bool refuses() const { return odd || least < (0x2dc00000u << 1) - 1u || !(most < 0.5f); }   // (2^-36)
    __device__ __forceinline__ void see(float x, float y)
    {
        const uint32_t ux = (__builtin_bit_cast(uint32_t, x) << 1) - 1u, uy = (__builtin_bit_cast(uint32_t, y) << 1) - 1u;
        least = min(least, min(ux, uy));
    }
    __device__ __forceinline__ void load(int krows)
    {
        if (tid < 256) {
            if (krows == BK) {
                if constexpr (transA) { pstage[0] = psrc[0]; pstage[1] = psrc[lda]; }
                else pstage = *(const f2_any *)psrc;
            } else {
                pstage[0] = pstage[1] = 0.0f;
                if (pk < krows) pstage[0] = psrc[0];
                if (pk + 1 < krows) pstage[1] = transA ? psrc[lda] : psrc[1];
            }
            psrc += transA ? (int64_t)BK * lda : BK;
        }
    }
    // A's pieces to LDS; B's staged values looked at and scaled
    template <int LOADS>
    __device__ __forceinline__ void store(int buf, f4v (&stage)[LOADS])
    {
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
    }
    // a stage's products on the matrix cores: the wave's 32 columns of B
    __device__ __forceinline__ void matrix_part(int buf)
    {
        const int li = lane & 31, lh = lane >> 5;
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
        constexpr int PA[6] = {2, 1, 1, 0, 0, 0}, PB[6] = {0, 0, 1, 1, 2, 0};     // (the largest last)
#pragma unroll
        for (int i = 0; i < 6; ++i)
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, ap[PA[i]]), __builtin_bit_cast(bf8, bp[PB[i]]), sum, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void dump()
    {
        const int li = lane & 31, lh = lane >> 5;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            L.s[8 * (v >> 2) + 4 * lh + (v & 3)][wave * 32 + li] = sum[v];
            sum[v] = 0.0f;
        }
    }
    __device__ __forceinline__ void fold(float (&part)[TM][4], float (&mainacc)[TM][4])
    {
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const f4v s4 = *(const f4v *)&L.s[wave * TM + r][lane * 4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // (what the addition rounds away starts the next partial sum)
                const float v = part[r][c] + s4[c], m = mainacc[r][c] + v;
                most = __builtin_fmaxf(most, part[r][c]);
                part[r][c] = v - (m - mainacc[r][c]);
                most = __builtin_fmaxf(most, __builtin_fabsf(part[r][c]));
                mainacc[r][c] = m;
            }
        }
    }
    // After a whole partial sum, where the stages so far are a power of two: what the waves have found, to be read by
    // all of them behind the next barrier
    __device__ __forceinline__ void tell()
    {
        const bool any = __builtin_amdgcn_ballot_w64(refuses()) != 0;
        if (lane == 0) L.refused[wave] = any;
    }
    __device__ __forceinline__ bool told() const
    {
        const u4 lo = *(const u4 *)&L.refused[0], hi = *(const u4 *)&L.refused[4], any = lo | hi;
        return __builtin_amdgcn_readfirstlane(any[0] | any[1] | any[2] | any[3]) != 0;
    }
};

// (what the kernel holds in the place of the pieces where there are none)
struct NoPieces {
    __device__ void load(int) {}
    template <typename Stage> __device__ void store(int, Stage &) {}
    __device__ void matrix_part(int) {}
    __device__ void dump() {}
    template <typename Acc, typename Main> __device__ void fold(Acc &, Main &) {}
    __device__ void tell() {}
    __device__ bool told() const { return false; }
};

}  // namespace amulet
#endif
