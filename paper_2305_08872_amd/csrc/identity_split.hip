// Identity task (g = p, plain matmul; paper Sec. 6.1) in fp32 on the bf16 matrix cores, for problems that fill the chip.
//
// An fp32 value is the sum of three bf16 pieces exactly: the value rounded to 8 significant bits, what that leaves
// (at most 16 bits) rounded to 8, and the rest.  A product of two values is then the sum of nine piece products, each exact in
// fp32, of which the six largest are formed here:
//     a b  =  a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0)  +  [a1 b2 + a2 b1 + a2 b2, left out]
// With |a1| <= 2^-8 |a| and |a2| <= 2^-17 |a| what is left out is random in sign, 3e-9 |a b| on average and 2^-24 |a b| at most
// (with a second piece that is cut, 9e-9 and 1.1e-7), beside the 2^-24 of an fp32 product's one rounding.
// v_mfma_f32_32x32x16_bf16 runs at sixteen times the rate of v_mfma_f32_32x32x2_f32 and rounds the accumulators once where that
// one does 8 times: six of them are faster, and over sums no less precise.  Relative error against 64 bits, fp32 matrix
// instructions / here with one set of accumulators / with two (below), uniform values: K = 96 1.8e-7 / 1.4e-7 / 5.3e-8, 256 2.9e-7 / 2.3e-7 /
// 8.1e-8, 1000 5.7e-7 / 4.8e-7 / 1.7e-7, 4096 1.15e-6 / - / 3.8e-7.  A product that stands alone in its sum -- A diagonal -- is rounded
// once by the fp32 instruction, 2.1e-8 of it on average and 6.0e-8 at most; here 2.7e-8 and 1.5e-7, with two sets 2.2e-8 and 9.6e-8.
//
// What bounds it is power: at 4096^3 the matrix cores are busy 65 % of the time at a clock that has fallen to some
// 1.75 GHz (the library's own bf16 product of that many operations runs at 1409 T/s, this kernel's six at 1140, with 256-row tiles
// at 1260).  With operands that change from call to call, fp32 matrix instructions / here: 4096^3 956 / 723 us (144 / 190 TFLOP/s; 128-row
// tiles: 256 rows take 654 there, see identity_split_wanted), 2048^3 129 / 108, 8192^2 x 1024 980 / 689 (256 rows).  Problems of fewer
// tiles gain nothing here (1024^3 with 64 x 64 tiles, in two designs, 24 us against 21 for the fp32 kernel): identity_split_waves.hip.
//
// Workgroup: 4 waves as 2 x 2, a wave WM x WN blocks of 32 x 32; two workgroups to a compute unit.  128 x 128 tiles with
// two sets of accumulators, one for a0 b0 and one for the five smaller products, whose roundings then count less; or 256 x
// 128, which read LDS and take values apart a quarter less per product and have registers for one set.  (A set
// per 16 k added up by the vector unit, 3.0e-7 at 4096^3, costs 14 % of the time.)  An operand's stage (16 k) goes global ->
// registers, DEPTH stages ahead -> pieces -> LDS, double buffered, one barrier per stage.  LDS keeps, per piece, [line][16
// k] in bf16 (line: a row of A, a column of B): a fragment read (lane: line l % 32, k = 8 (l / 32) .. + 7) is 64 lanes times 16
// contiguous bytes, and so is a write: no bank conflicts.
//
// Values that the pieces do not carry: one with bits below 2^-133, the least a bf16 has (any below 2^-109 may), leaves a
// remainder, whose low half is not zero; a NaN or infinity (also a finite value that rounds to an infinite
// bf16) leaves a NaN in the accumulators.  A workgroup that finds a NaN at its end, or a remainder there or in its
// first stage, forms its tile again with the fp32 matrix instruction (fp32_sums).  us, none of these / all values / one, or an
// infinity / one in every tile / the fp32 kernels: 2048^3 106 / 169 / 256 / 260 / 128, 4096^3 705 / 1098 / 931 / 1800 / 943, 3000 x 5000 x 1000
// 165 / 274 / 285 / 424 / 247.  (From global memory, a matrix instruction for every 2 k, as this once was: 2048^3 one 593, all 549,
// 4096^3 1496, 2710, B transposed 4103.  Looks during the loop, after 8, 16, 32 ... stages, cost 4096^3 0.5 to 1 % wherever they stood.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amulet_internal.h"
#include "pieces.h"

namespace amulet {

typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <int WM, int WN>
struct SplitTile {
    static constexpr int BM = 64 * WM, BN = 64 * WN, BK = 16;
    static constexpr int A_PIECE = BM * 32, B_PIECE = BN * 32;                 // bytes of a piece in a stage
    static constexpr int A_BYTES = 3 * A_PIECE, STAGE_BYTES = A_BYTES + 3 * B_PIECE;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES + 16;                     // (and a word per wave: what it has found)
    static constexpr int UA = BM / 128, UB = BN / 128;                         // units (8 k of a line) per thread
    static constexpr int NACC = WM * WN >= 8 ? 1 : 2;                          // accumulator sets
    static constexpr int DEPTH = WM * WN >= 8 ? 1 : 2;                         // stages in flight in registers (a fuller wave has fewer left)
};

extern __shared__ __attribute__((aligned(16))) char split_smem[];

// One operand's way from memory to the pieces: U units of 8 k of a line per thread, unit = tid + 256 j: line
// unit / 2, k half unit % 2.
template <int U, int DEPTH, bool KMINOR>
struct Operand {
    static constexpr int PIECE = U * 128 * 32;
    const float *base, *end;   // the tile's first line at the next stage to load; past the operand's last value
    int64_t ld;
    uint32_t off[U];           // bytes from `base` to the unit's first value
    uint32_t left_over;        // OR of what the pieces left
    float x[DEPTH][U][8];      // raw values of the next DEPTH stages
    u4 piece[3];               // of the unit being taken apart

    // `first`: the tile's first line at k = 0 of `k`; `lines` of the operand from it on
    __device__ __forceinline__ void start(const float *first, int64_t pitch, int lines, int k, int tid)
    {
        base = first;
        ld = pitch;
        end = KMINOR ? first + (int64_t)(lines - 1) * pitch + k : first + (int64_t)(k - 1) * pitch + lines;
        left_over = 0;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int line = (tid + 256 * j) >> 1, in = line < lines ? line : lines - 1;   // (past the edge: the last line inside)
            const uint32_t k0 = (uint32_t)(tid & 1) * 8u;
            off[j] = KMINOR ? ((uint32_t)in * (uint32_t)ld + k0) * 4u : (k0 * (uint32_t)ld + (uint32_t)in) * 4u;
        }
    }
    // Unit j of the stage at `base` into ring slot d.  One address register per unit: the base is scalar, and so
    // is the row of a k-major operand in the offset of a buffer load (which also keeps a stage's rows inside the operand).
    __device__ __forceinline__ void load(int d, int j)
    {
        if constexpr (KMINOR) {
            const f4 v0 = *(const f4 *)((const char *)base + off[j]), v1 = *(const f4 *)((const char *)base + off[j] + 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[d][j][i] = v0[i]; x[d][j][4 + i] = v1[i]; }
        } else {
            const int64_t bytes = (const char *)end - (const char *)base;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, bytes < 0x7fffffff ? (int)bytes : 0x7fffffff, 0x00027000);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[d][j][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[j], i * (int)ld * 4, 0));
        }
    }
    // zeros for the k past a short stage's `left`
    __device__ __forceinline__ void cut(int d, int j, int tid, int left)
    {
        const int k0 = (tid & 1) * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[d][j][i] = k0 + i < left ? x[d][j][i] : 0.0f;
    }
    // unit j of ring slot 0 into LDS as it is: [k / 4][line][4 k]
    __device__ __forceinline__ void put(int j, int tid, char *lds)
    {
        const int line = (tid + 256 * j) >> 1, quad = (tid & 1) * 2;
        *(f4 *)(lds + (quad * U * 128 + line) * 16) = f4{x[0][j][0], x[0][j][1], x[0][j][2], x[0][j][3]};
        *(f4 *)(lds + ((quad + 1) * U * 128 + line) * 16) = f4{x[0][j][4], x[0][j][5], x[0][j][6], x[0][j][7]};
    }
    __device__ __forceinline__ void advance(int k) { base += KMINOR ? (int64_t)k : (int64_t)k * ld; }
    // pair i of unit j into pieces; after the fourth, the unit into LDS
    __device__ __forceinline__ void take(int d, int j, int i, int tid, char *lds)
    {
        uint32_t p0, p1, p2;
        left_over |= take_pieces(x[d][j][2 * i], x[d][j][2 * i + 1], p0, p1, p2);
        piece[0][i] = p0; piece[1][i] = p1; piece[2][i] = p2;
        if (i == 3) {
#pragma unroll
            for (int q = 0; q < 3; ++q) *(u4 *)(lds + q * PIECE + (tid + 256 * j) * 16) = piece[q];
        }
    }
};

// The tile's sums on the fp32 matrix cores, whatever the values: a stage of 16 k in registers, one in LDS, one being multiplied.
// A lane's fragment is 8 k in a row of its line, those of the lanes 32 on the other 8: a matrix instruction's two k are 8 apart.
template <int WM, int WN, bool TA, bool TB, typename Args>
__device__ __forceinline__ void fp32_sums(const Args &args, const int tid, const int row0, const int col0, f16v (&acc)[WM][WN])
{
    typedef SplitTile<WM, WN> TL;
    constexpr int BK = TL::BK, UA = TL::UA, UB = TL::UB, A_BYTES = TL::BM * BK * 4, BYTES = A_BYTES + TL::BN * BK * 4;
    static_assert(2 * BYTES <= TL::LDS_BYTES, "two stages in the pieces' LDS");
    const int K = args.K, n_stages = (K + BK - 1) / BK, first_k = K - (n_stages - 1) * BK;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1, li = lane & 31, lh = lane >> 5;
    Operand<UA, 1, !TA> a;
    Operand<UB, 1, TB> b;
    a.start(TA ? args.A + row0 : args.A + (int64_t)row0 * args.lda, args.lda, args.M - row0, K, tid);
    b.start(TB ? args.B + (int64_t)col0 * args.ldb : args.B + col0, args.ldb, args.N - col0, K, tid);
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < UA; ++u) a.load(0, u);
#pragma unroll
        for (int u = 0; u < UB; ++u) b.load(0, u);
    };
    auto put = [&](char *lds) {
#pragma unroll
        for (int u = 0; u < UA; ++u) a.put(u, tid, lds);
#pragma unroll
        for (int u = 0; u < UB; ++u) b.put(u, tid, lds + A_BYTES);
    };
    load();
#pragma unroll
    for (int u = 0; u < UA; ++u) a.cut(0, u, tid, first_k);
#pragma unroll
    for (int u = 0; u < UB; ++u) b.cut(0, u, tid, first_k);
    put(split_smem);
    if (n_stages > 1) { a.advance(first_k); b.advance(first_k); }
    load();
#pragma unroll
    for (int mi = 0; mi < WM; ++mi)
#pragma unroll
        for (int ni = 0; ni < WN; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < n_stages; ++s) {
        const char *lds = split_smem + (s & 1) * BYTES;
        f4 af[WM][2], bf[WN][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int mi = 0; mi < WM; ++mi) af[mi][h] = *(const f4 *)(lds + ((2 * lh + h) * TL::BM + (wr * WM + mi) * 32 + li) * 16);
#pragma unroll
            for (int ni = 0; ni < WN; ++ni) bf[ni][h] = *(const f4 *)(lds + A_BYTES + ((2 * lh + h) * TL::BN + (wc * WN + ni) * 32 + li) * 16);
        }
        // (past the last stage: the last one again, which nothing reads)
        put(split_smem + ((s + 1) & 1) * BYTES);
        if (s + 2 < n_stages) { a.advance(BK); b.advance(BK); }
        load();
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int mi = 0; mi < WM; ++mi)
#pragma unroll
                for (int ni = 0; ni < WN; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi][k / 4][k % 4], bf[ni][k / 4][k % 4], acc[mi][ni], 0, 0, 0);
        __syncthreads();
    }
}

template <int WM, int WN, bool TA, bool TB>
__global__ void __launch_bounds__(256, 2) identity_split_kernel(const MmlikeArgs args)
{
    typedef SplitTile<WM, WN> TL;
    constexpr int BM = TL::BM, BN = TL::BN, BK = TL::BK;
    const int M = args.M, N = args.N;
    const int K = args.K;   // (at least a stage, the host checks)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1, li = lane & 31, lh = lane >> 5;

    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, tiles_m, tiles_n, tm, tn)) return;   // padding: the whole workgroup leaves
    const int row0 = __builtin_amdgcn_readfirstlane(tm * BM), col0 = __builtin_amdgcn_readfirstlane(tn * BN);
    const int rows_in = M - row0 < BM ? M - row0 : BM, cols_in = N - col0 < BN ? N - col0 : BN;
    const int n_stages = (K + BK - 1) / BK, first_k = K - (n_stages - 1) * BK;

    constexpr int DEPTH = TL::DEPTH, UA = TL::UA, UB = TL::UB;
    Operand<UA, DEPTH, !TA> a;
    Operand<UB, DEPTH, TB> b;
    a.start(TA ? args.A + row0 : args.A + (int64_t)row0 * args.lda, args.lda, M - row0, K, tid);
    b.start(TB ? args.B + (int64_t)col0 * args.ldb : args.B + col0, args.ldb, N - col0, K, tid);

    // (NACC = 2: the five smaller products of a step have accumulators of their own, which round in proportion to them)
    constexpr int NACC = TL::NACC;
    f16v sums[NACC][WM][WN];
#pragma unroll
    for (int c = 0; c < NACC; ++c)
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int ni = 0; ni < WN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) sums[c][mi][ni][v] = 0.0f;

    // unit u of a stage (A's first) into ring slot d, and from there, pair by pair, into an LDS buffer
    int loaded = 1;
    auto load = [&](int d, int u) {
        if (u < UA) a.load(d, u);
        else b.load(d, u - UA);
        if (u == UA + UB - 1 && ++loaded < n_stages) { a.advance(BK); b.advance(BK); }   // (past the last stage: the last one again)
    };
    auto take = [&](int d, int u, int i, char *lds) {
        if (u < UA) a.take(d, u, i, tid, lds);
        else b.take(d, u - UA, i, tid, lds + TL::A_BYTES);
    };
    const int a_frag = (wr * 32 * WM + li) * 32 + lh * 16, b_frag = TL::A_BYTES + (wc * 32 * WN + li) * 32 + lh * 16;
    bf8 af[3][WM], bf[3][WN];
    auto read_a = [&](const char *lds, int q) {
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) af[q][mi] = *(const bf8 *)(lds + a_frag + q * TL::A_PIECE + mi * 1024);
    };
    auto read_b = [&](const char *lds, int q) {
#pragma unroll
        for (int ni = 0; ni < WN; ++ni) bf[q][ni] = *(const bf8 *)(lds + b_frag + q * TL::B_PIECE + ni * 1024);
    };

    // Stage 0 to LDS, the next DEPTH on their way.  Where K is not whole stages, stage 0 is the short one.
#pragma unroll
    for (int u = 0; u < UA; ++u) { a.load(0, u); a.cut(0, u, tid, first_k); }
#pragma unroll
    for (int u = 0; u < UB; ++u) { b.load(0, u); b.cut(0, u, tid, first_k); }
    if (n_stages > 1) { a.advance(first_k); b.advance(first_k); }
#pragma unroll
    for (int u = 0; u < UA + UB; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) take(0, u, i, split_smem);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
#pragma unroll
        for (int u = 0; u < UA + UB; ++u) load(d, u);
    // (where stage 0 already has values that the pieces do not carry, as operands full of them have, no further one is begun)
    uint32_t *const found = (uint32_t *)(split_smem + 2 * TL::STAGE_BYTES);
    const bool any = __builtin_amdgcn_ballot_w64(((a.left_over | b.left_over) & 0xffffu) != 0) != 0;
    if (lane == 0) found[wave] = any;
    __syncthreads();
    const u4 told = *(const u4 *)found;
    const int stages = __builtin_amdgcn_readfirstlane(told[0] | told[1] | told[2] | told[3]) != 0 ? 0 : n_stages;
    read_a(split_smem, 1);
    read_b(split_smem, 1);

    // One stage.  The six piece products in an order in which few pieces are live at a time, the fragments read a
    // product ahead; between the matrix instructions (some six vector instructions to each run in its shade) the next
    // stage's values are taken apart and written to the other buffer, and a unit's registers reloaded DEPTH stages
    // ahead (past the last stage: that one again, which nothing reads).  The barrier stands before the stage's last product: by
    // then this wave has read all of the stage and written all of the next, and behind it are matrix
    // instructions enough to cover the first reads of the next.
    auto stage = [&](int s, int d) {
        char *lds = split_smem + (s & 1) * TL::STAGE_BYTES, *other = split_smem + ((s + 1) & 1) * TL::STAGE_BYTES;
        constexpr int PA[6] = {1, 1, 2, 0, 0, 0}, PB[6] = {1, 0, 0, 1, 2, 0};     // (the largest last: a product that stands alone is rounded once)
        constexpr int BLOCKS = WM * WN, NM = 5 * BLOCKS, PAIRS = 4 * (UA + UB);   // (nothing to take apart during the last product)
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) {
            if (pq == 0) read_b(lds, 0);
            else if (pq == 1) read_a(lds, 2);
            else if (pq == 2) read_a(lds, 0);
            else if (pq == 3) read_b(lds, 2);
            else if (pq == 5) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();   // bare: the fence of __syncthreads() would drain the loads in flight
                asm volatile("" ::: "memory");
                read_a(other, 1);
                read_b(other, 1);
            }
#pragma unroll
            for (int m = 0; m < BLOCKS; ++m) {
                const int mi = m / WN, ni = m % WN;
                f16v &sum = sums[PA[pq] + PB[pq] == 0 ? 0 : NACC - 1][mi][ni];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[PA[pq]][mi], bf[PB[pq]][ni], sum, 0, 0, 0);
                const int at = pq * BLOCKS + m;
                if (at < NM) {
#pragma unroll
                    for (int p = (at * PAIRS + NM - 1) / NM; p < PAIRS && p * NM < (at + 1) * PAIRS; ++p) {
                        take(d, p / 4, p % 4, other);
                        if (p % 4 == 3) load(d, p / 4);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if constexpr (DEPTH == 1) {
        for (int s = 0; s < stages; ++s) stage(s, 0);
    } else {
        int s = 0;
        for (; s + 1 < stages; s += 2) { stage(s, 0); stage(s + 1, 1); }
        if (s < stages) stage(s, 0);
    }

    f16v (&acc)[WM][WN] = sums[0];
    if constexpr (NACC == 2) {
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int ni = 0; ni < WN; ++ni) acc[mi][ni] += sums[1][mi][ni];
    }
    // pieces that do not carry their values: once more, in fp32
    bool again = ((a.left_over | b.left_over) & 0xffffu) != 0;
#pragma unroll
    for (int mi = 0; mi < WM; ++mi)
#pragma unroll
        for (int ni = 0; ni < WN; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) again |= !(__builtin_fabsf(acc[mi][ni][v]) <= 3.402823466e+38f);
    if (__syncthreads_or(again)) {
        unsigned t;
        const auto &same = opaque_args<MmlikeArgs>(wave, t);
        fp32_sums<WM, WN, TA, TB>(same, (int)t, row0, col0, acc);
    }

    // accumulator element v of lane l is R[8*(v/4) + 4*(l/32) + v%4][l%32] of its 32 x 32 block; a row of
    // blocks is read whole before the first sum is stored.  An edge tile adds with atomics, the elements that exist (R
    // has one owner, the sum is the same single rounding, and no load waits under a mask).
    const bool edge = rows_in < BM || cols_in < BN;
#pragma unroll
    for (int mi = 0; mi < WM; ++mi) {
        const int row = (wr * WM + mi) * 32 + 4 * lh, col = wc * WN * 32 + li;
        float *dst = args.R + (int64_t)(row0 + row) * args.ldr + col0 + col;
        if (edge) {
#pragma unroll
            for (int ni = 0; ni < WN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (row + 8 * (v >> 2) + (v & 3) < rows_in && col + 32 * ni < cols_in)
                        unsafeAtomicAdd(dst + (int64_t)(8 * (v >> 2) + (v & 3)) * args.ldr + 32 * ni, acc[mi][ni][v]);
        } else {
            float old[WN][16];
#pragma unroll
            for (int ni = 0; ni < WN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) old[ni][v] = dst[(int64_t)(8 * (v >> 2) + (v & 3)) * args.ldr + 32 * ni];
#pragma unroll
            for (int ni = 0; ni < WN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[(int64_t)(8 * (v >> 2) + (v & 3)) * args.ldr + 32 * ni] = old[ni][v] + acc[mi][ni][v];
        }
    }
}

template <int WM, int WN, bool TA, bool TB>
static hipError_t launch_layout(MmlikeArgs &a, int64_t grid, hipStream_t s)
{
    constexpr int LDS = SplitTile<WM, WN>::LDS_BYTES;
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&identity_split_kernel<WM, WN, TA, TB>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (granted != hipSuccess) return granted;
    return launch_row_of_blocks(a, grid, 256, [&](unsigned n) {
        hipLaunchKernelGGL((identity_split_kernel<WM, WN, TA, TB>), dim3(n), dim3(256), LDS, s, a);
    });
}

template <int WM, int WN>
static hipError_t launch_tile(MmlikeArgs &a, int64_t grid, hipStream_t s)
{
    if (a.transA && a.transB) return launch_layout<WM, WN, true, true>(a, grid, s);
    if (a.transA) return launch_layout<WM, WN, true, false>(a, grid, s);
    if (a.transB) return launch_layout<WM, WN, false, true>(a, grid, s);
    return launch_layout<WM, WN, false, false>(a, grid, s);
}

// A stage of K, and per-lane byte offsets that fit 31 bits (a k-minor stage spans up to 256 lines of an operand's
// storage, a k-major one 16); every other size, and every alignment, runs.
bool identity_split_runs(bool trans_a, bool trans_b, int64_t K, int64_t lda, int64_t ldb)
{
    const int64_t minor_max = (0x7FFFFFFFLL / 4 - 16) / 256, major_max = (0x7FFFFFFFLL / 4 - 256) / 16;
    return K >= 16 && lda <= (trans_a ? major_max : minor_max) && ldb <= (trans_b ? minor_max : major_max);
}

hipError_t launch_identity_split(const MmlikeArgs &a, int tile_rows, hipStream_t s)
{
    MmlikeArgs b = a;
    const int64_t grid = xcd_grid(((int64_t)a.M + tile_rows - 1) / tile_rows, ((int64_t)a.N + 127) / 128);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    if (tile_rows == 256) return launch_tile<4, 2>(b, grid, s);
    return launch_tile<2, 2>(b, grid, s);
}

}  // namespace amulet
