// BOOST with its two sums on two units (boost_pieces.h): the wide kernel in that form, and its launch.
#include "mmlike_valu_impl.h"

#ifndef AMULET_MMLIKE_BOOST_IMPL_H
#define AMULET_MMLIKE_BOOST_IMPL_H

namespace amulet {

// A workgroup's work on its tile, by pieces or by the wide kernel's own arithmetic.  False: the tile holds values that the
// pieces do not take, and R is as it was.
template <int TF, int TRANS, bool PIECES, typename Args>
__device__ __forceinline__ bool boost_tile(const Args &args, const unsigned tid, BoostLds &L)
{
    constexpr int TASK = TASK_BOOST, TM = 4, NG = 1, NW = 8, BK = BOOST_BK, KA = 4;
    constexpr bool ALDS = false, PIPE = false, BPRE = (TRANS & 1) == 0;
    auto &Bs = L.b;
    auto &Asl = *(float (*)[1][1][4])L.s;
    auto done = [](bool whole) { return whole; };
#include "mmlike_valu_tile.inc"
}

// A tile that has to be formed again is, from the start, with nothing of the first way in registers: the kernel's arguments and
// the thread's number are opaque there, or what both ways compute alike is held through the first's loop (42 registers too many).
template <int TF, int TRANS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
mmlike_boost_kernel(const MmlikeArgs args)
{
    extern __shared__ __attribute__((aligned(16))) char boost_smem[];
    BoostLds &L = *(BoostLds *)boost_smem;
    if (__builtin_expect(boost_tile<TF, TRANS, true>(args, threadIdx.x, L), true)) return;
    auto at = (const __attribute__((address_space(4))) MmlikeArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    unsigned tid = threadIdx.x;
    asm volatile("" : "+s"(at), "+v"(tid));
    boost_tile<TF, TRANS, false>(*at, tid, L);
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
