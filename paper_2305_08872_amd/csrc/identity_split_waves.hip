// Identity task in fp32 from bf16 pieces (identity_split.hip, which says what they are and what they cost in precision) for problems of
// few tiles: the waves of a workgroup share K.
//
// Workgroup: a tile of 64 x 64, eight waves, each of which forms all of it over an eighth of K and meets the others in LDS at the end. A
// wave streams its 16 k of 64 rows and 64 columns HBM -> LDS of its own (two stages, 8 KiB each; no barrier before the end), takes
// them apart in registers and runs 24 matrix instructions on them, while the other wave of its SIMD takes its own apart. Two sets of
// accumulators, of an eighth of K each: relative error over uniform values at K = 1024 8.2e-8, fp32 matrix instructions 4.1e-7.
//
// What bounds it: at 1024^3 the six products take 9.3 us of the 18.4 with nothing loaded (1385 T/s in bf16, what the power allows), 11.4
// with loads; the rest is the launch and both ends. us, the fp32 kernel's 64 x 64 tiles / here: 1024^3 20.7 / 18.4, 1018 x 1004 x 3347 60.4 / 51.1,
// 531 x 1600 x 3705 60.0 / 47.4, 2240 x 297 x 1216, both transposed, 26.2 / 19.6, 1280 x 1536 x 2215, both transposed, 71.4 / 62.1; short K or few tiles
// not (512^3 7.9 / 10.0, 1024^2 x 256 8.2 / 9.0). Measured and not kept: fragments of an operand stored along k straight from memory, 32 rows by 16 bytes
// a load (1024^3 20.9; across k, 128 bytes of 32 columns, 17.2, as fast as through LDS); one set of accumulators and the next step's values
// taken apart between the matrix instructions (19.9); loads through registers two steps ahead (spills).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amulet_internal.h"
#include <type_traits>

#include "pieces.h"

// the LDS-DMA asm below sets M0 itself and says so in its clobber list
#pragma clang diagnostic ignored "-Winline-asm"

namespace amulet {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef f4 f4_any __attribute__((aligned(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_void_ptr;

constexpr int SW_TILE = 64, SW_WAVES = 8, SW_BK = 16;
constexpr int SW_PITCH = SW_TILE + 4;

extern __shared__ __attribute__((aligned(16))) float sw_sums[];      // a tile of sums per wave

// A wave's 64 lines (rows of A, columns of B) by 16 k: HBM -> LDS of the wave's own, and from there its two fragments: lane l has 8 k from
// 8 (l / 32) on of line l % 32 and of the 32nd after it.  LDS holds an operand as it is stored: 64 bytes per line, or 256 per k; a
// unit of 16 bytes at a place that spreads the reads over the banks.  A line past the edge is the last one inside; a unit across
// k that the edge cuts is the four lines that end there.
template <bool KMINOR>
struct WaveOperand {
    const float *base;
    int64_t ld;
    uint32_t off[4];       // bytes from a stage's first value to the lane's unit of kilobyte j
    uint32_t at[2];        // a lane's first value of fragment j in the stage's LDS

    // `first`: the tile's first line; `lines` of the operand from there on.  (Across k, with fewer than four of them: from the operand's
    // last four on.)
    __device__ __forceinline__ void start(const float *first, int64_t pitch, int lines, int lane)
    {
        const int back = !KMINOR && lines < 4 ? 4 - lines : 0;
        base = first - back;
        ld = pitch;
        lines += back;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (KMINOR) {
                const int line = (lane >> 2) + 16 * j, in = line < lines ? line : lines - 1;
                off[j] = ((uint32_t)in * (uint32_t)ld + (uint32_t)((lane & 3) ^ ((line >> 2) & 3)) * 4u) * 4u;
            } else {
                const int k = (lane >> 4) + 4 * j, line = ((lane & 15) ^ (k & 8)) * 4 + back, in = line < lines - 4 ? line : lines - 4;
                off[j] = (uint32_t)(k * (int)ld + in) * 4u;
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int line = (lane & 31) + 32 * j, lh = lane >> 5;
            if constexpr (KMINOR) at[j] = (uint32_t)(line * 64 + ((2 * lh) ^ ((line >> 2) & 3)) * 16);
            else {
                const int unit = line >> 2, own = unit * 4 + back, from = own < lines - 4 ? own : lines - 4, e = line + back - from < 4 ? line + back - from : 3;
                at[j] = (uint32_t)(lh * 8 * 256 + (unit ^ (lh * 8)) * 16 + e * 4);
            }
        }
    }
    __device__ __forceinline__ const float *stage(int k) const { return base + (KMINOR ? (int64_t)k : (int64_t)k * ld); }
    __device__ __forceinline__ void read(float (&y)[2][8], const char *lds) const
    {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (KMINOR) {
                const f4 v0 = *(const f4 *)(lds + at[j]), v1 = *(const f4 *)(lds + (at[j] ^ 16u));
#pragma unroll
                for (int i = 0; i < 4; ++i) { y[j][i] = v0[i]; y[j][4 + i] = v1[i]; }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) y[j][i] = *(const float *)(lds + at[j] + i * 256);
            }
        }
    }
};

template <bool TA, bool TB>
__global__ void __launch_bounds__(64 * SW_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
identity_split_waves_kernel(const MmlikeArgs args)
{
    const int M = args.M, N = args.N, K = args.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_m = (M + SW_TILE - 1) / SW_TILE, tiles_n = (N + SW_TILE - 1) / SW_TILE;
    int tm, tn;
    if (!xcd_tile((int)blockIdx.x + args.block_base, tiles_m, tiles_n, tm, tn)) return;
    const int row0 = tm * SW_TILE, col0 = tn * SW_TILE;
    // a wave's k: an eighth, in whole steps
    const int share = ((K + SW_WAVES - 1) / SW_WAVES + SW_BK - 1) / SW_BK * SW_BK;
    const int first = wave * share, left = K - first, len = left < 0 ? 0 : left < share ? left : share;
    const int steps = (len + SW_BK - 1) / SW_BK;

    f16v sums[2][2][2];
    auto clear = [&] {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sums[c][mi][ni][v] = 0.0f;
    };
    clear();
    WaveOperand<!TA> a;
    WaveOperand<TB> b;
    a.start(TA ? args.A + row0 : args.A + (int64_t)row0 * args.lda, args.lda, M - row0, lane);
    b.start(TB ? args.B + (int64_t)col0 * args.ldb : args.B + col0, args.ldb, N - col0, lane);
    // step s: the 16 k from first + 16 s on, or, where fewer are left, the last 16 there are, cut to those
    auto window = [&](int s) { const int k = first + s * SW_BK; return k < K - SW_BK ? k : K - SW_BK; };
    const char *const own = (const char *)(sw_sums + wave * (SW_TILE * SW_PITCH));
    const uint32_t own_lds = (uint32_t)(uintptr_t)(lds_void_ptr)sw_sums + (uint32_t)wave * (SW_TILE * SW_PITCH * 4);
    auto issue = [&](int s) {      // (past the last step: that one again, which nothing reads)
        const int k = window(s < steps ? s : steps - 1);
        const float *pa = a.stage(k), *pb = b.stage(k);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(own_lds + (uint32_t)(s & 1) * 8192u);
#define SW_LOAD(V, P, O) "s_add_u32 m0, %[d], " #O "\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[" #V "], %[" #P "]\n\t"
        asm volatile(SW_LOAD(a0, a, 0) SW_LOAD(a1, a, 0x400) SW_LOAD(a2, a, 0x800) SW_LOAD(a3, a, 0xc00)
                     SW_LOAD(b0, b, 0x1000) SW_LOAD(b1, b, 0x1400) SW_LOAD(b2, b, 0x1800) SW_LOAD(b3, b, 0x1c00)
                     :: [d] "s"(dst), [a] "s"(pa), [b] "s"(pb), [a0] "v"(a.off[0]), [a1] "v"(a.off[1]), [a2] "v"(a.off[2]), [a3] "v"(a.off[3]),
                        [b0] "v"(b.off[0]), [b1] "v"(b.off[1]), [b2] "v"(b.off[2]), [b3] "v"(b.off[3]) : "memory", "m0", "scc");
#undef SW_LOAD
    };
    uint32_t left_over = 0;
    auto cut = [&](float (&y)[2][8], int gone) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) y[j][i] = (lane >> 5) * 8 + i >= gone ? y[j][i] : 0.0f;
    };
    auto take = [&](const float (&x)[2][8], bf8 (&p)[3][2]) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            u4 w[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t p0, p1, p2;
                left_over |= take_pieces(x[j][2 * i], x[j][2 * i + 1], p0, p1, p2);
                w[0][i] = p0; w[1][i] = p1; w[2][i] = p2;
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) p[q][j] = __builtin_bit_cast(bf8, w[q]);
        }
    };
    auto all_steps = [&](auto fp32) {
        if (steps == 0) return;
        issue(0);
        issue(1);
#pragma unroll 1
        for (int s = 0; s < steps; ++s) {
            float ya[2][8], yb[2][8];
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            const char *lds = own + (s & 1) * 8192;
            a.read(ya, lds);
            b.read(yb, lds + 4096);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            issue(s + 2);
            const int gone = first + s * SW_BK - window(s);
            if (gone > 0) { cut(ya, gone); cut(yb, gone); }
            if constexpr (decltype(fp32)::value) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                        for (int ni = 0; ni < 2; ++ni) sums[0][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(ya[mi][i], yb[ni][i], sums[0][mi][ni], 0, 0, 0);
            } else {
                bf8 pa[3][2], pb[3][2];
                take(ya, pa);
                take(yb, pb);
                constexpr int PA[6] = {1, 1, 2, 0, 0, 0}, PB[6] = {1, 0, 0, 1, 2, 0};
#pragma unroll
                for (int pq = 0; pq < 6; ++pq)
#pragma unroll
                    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                        for (int ni = 0; ni < 2; ++ni) {
                            f16v &sum = sums[PA[pq] + PB[pq] == 0 ? 0 : 1][mi][ni];
                            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[PA[pq]][mi], pb[PB[pq]][ni], sum, 0, 0, 0);
                        }
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    all_steps(std::false_type());
    f16v (&acc)[2][2] = sums[0];
    bool again = (left_over & 0xffffu) != 0;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            acc[mi][ni] += sums[1][mi][ni];
#pragma unroll
            for (int v = 0; v < 16; ++v) again |= !(__builtin_fabsf(acc[mi][ni][v]) <= 3.402823466e+38f);
        }
    // (a wave's part by itself: the pieces do not carry its values, once more with the fp32 instruction)
    if (__builtin_amdgcn_ballot_w64(again) != 0) {
        clear();
        all_steps(std::true_type());
    }
    // The waves' sums meet in LDS, by columns: accumulator element v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of its
    // 32 x 32 block, four rows to a 16-byte write.
    const int li = lane & 31, lh = lane >> 5;
    float *const mine = sw_sums + wave * (SW_TILE * SW_PITCH);
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f4 *)(mine + (ni * 32 + li) * SW_PITCH + mi * 32 + 8 * q + 4 * lh) = f4{acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]};
    // a thread's eight outputs: rows 8 wave .. + 7 of column `lane`
    const int row = row0 + wave * 8, col = col0 + lane, rows = M - row < 8 ? M - row : 8;
    float *const dst = args.R + (int64_t)row * args.ldr + col;
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = col < N && i < rows ? dst[(int64_t)i * args.ldr] : 0.0f;
    __syncthreads();
    f4 sum[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        sum[h] = *(const f4 *)(sw_sums + lane * SW_PITCH + wave * 8 + 4 * h);
#pragma unroll
        for (int w = 1; w < SW_WAVES; ++w) sum[h] += *(const f4 *)(sw_sums + w * (SW_TILE * SW_PITCH) + lane * SW_PITCH + wave * 8 + 4 * h);
    }
    if (col < N)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < rows) dst[(int64_t)i * args.ldr] = r[i] + sum[i >> 2][i & 3];
}

template <bool TA, bool TB>
static hipError_t launch_waves(const MmlikeArgs &args, hipStream_t s)
{
    constexpr int LDS = SW_WAVES * SW_TILE * SW_PITCH * 4;
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&identity_split_waves_kernel<TA, TB>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (granted != hipSuccess) return granted;
    MmlikeArgs a = args;
    const int64_t grid = xcd_grid(((int64_t)a.M + SW_TILE - 1) / SW_TILE, ((int64_t)a.N + SW_TILE - 1) / SW_TILE);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    return launch_row_of_blocks(a, grid, 64 * SW_WAVES, [&](unsigned n) {
        hipLaunchKernelGGL((identity_split_waves_kernel<TA, TB>), dim3(n), dim3(64 * SW_WAVES), LDS, s, a);
    });
}

hipError_t launch_identity_split_waves(const MmlikeArgs &a, hipStream_t s)
{
    if (a.transA && a.transB) return launch_waves<true, true>(a, s);
    if (a.transA) return launch_waves<true, false>(a, s);
    if (a.transB) return launch_waves<false, true>(a, s);
    return launch_waves<false, false>(a, s);
}

}  // namespace amulet
